"""KeyGen, staged Sign and Verify at the counts where their hash chains go from a wavefront per state to a
16-lane row, a lane pair or a lane (2048 / 4096 / 8192 states; a Sign task has l mask streams), with
messages that end before, at and after a block edge.  Everything equals the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2211_12265_amd import workload

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("level,count", [(2, 1), (2, 512), (2, 513), (3, 819), (3, 820), (44, 1024), (44, 1025),
                                         (87, 2048), (65, 2049), (5, 4096), (2, 4097), (44, 8193)])
def test_counts_where_states_change(level, count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_12265_amd import dilithium as dl
    pkl, skl, sgl = dl.sizes(level)
    seeds = workload.keygen_seeds(count, seed=900 + level)
    opk, osk = oracle.keygen_batch(level, seeds)
    lens = (np.array([0, 1, 69, 70, 71, 72, 73, 103, 104, 105, 136, 205, 208, 344])[np.arange(count) % 14])
    msg, off = workload.messages(lens, seed=count)
    osig, _ = oracle.sign_batch(level, osk, msg, off)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    new = lambda w: torch.zeros((count, w), dtype=torch.uint8, device="cuda")
    ctx = dl.Context(0, mode=dl.MODE_STAGED)
    pk, sk, sig = new(pkl), new(skl), new(sgl)
    ctx.keygen(level, dev(seeds), pk, sk)
    assert np.array_equal(pk.cpu().numpy(), opk) and np.array_equal(sk.cpu().numpy(), osk)
    dmsg, doff = dev(msg), dev(off.astype(np.int64))
    ctx.sign(level, sk, dmsg, doff, sig)
    torch.cuda.synchronize()
    assert np.array_equal(sig.cpu().numpy(), osig)
    bad = sig.clone()
    rows = torch.arange(0, count, 3, device="cuda")
    bad[rows, rows % sgl] ^= 1                       # each byte of a signature in some task
    ok = torch.full((count,), 9, dtype=torch.int32, device="cuda")
    ctx.verify(level, pk, dmsg, doff, bad, ok)
    torch.cuda.synchronize()
    want = np.ones(count, dtype=np.int32)
    want[::3] = 0
    assert np.array_equal(ok.cpu().numpy(), want)
    ctx.close()
