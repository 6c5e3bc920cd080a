"""Key-table Verify at the count where its hash chains and main part go from one launch to three (1024
tasks), through both entry points, with messages of 0 .. 400 bytes and a flipped byte in every third
signature (each place in some task)."""
import numpy as np
import pytest

import oracle
from paper_2211_12265_amd import workload

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("level,count", [(2, 1), (65, 7), (2, 1024), (44, 1025), (87, 1024), (5, 1025)])
def test_one_launch_or_three(level, count, noalloc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_12265_amd import dilithium as dl
    nk = min(count, 19)
    pk, sk = oracle.keygen_batch(level, workload.keygen_seeds(nk, seed=970 + level))
    key_idx = (np.arange(count) * 7 % nk).astype(np.uint32)
    msg, off = workload.messages(workload.uniform_lengths(count, 0, 400, seed=count), seed=count)
    sig, _ = oracle.sign_batch(level, sk, msg, off, key_idx=key_idx)
    sig = sig.copy()
    rows = np.arange(0, count, 3)
    sig[rows, (rows * 37) % sig.shape[1]] ^= 0x40
    want = np.ones(count, dtype=np.int32)
    want[rows] = 0
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ctx = dl.Context(0)
    ks = dl.KeySet(ctx, level, pk=dev(pk))
    ok = torch.full((count,), 9, dtype=torch.int32, device="cuda")
    for _ in range(2):   # the second call replays what the first recorded
        ks.verify(ctx, dev(key_idx.astype(np.int32)), dev(msg), dev(off.astype(np.int64)), dev(sig), ok,
                  noalloc=noalloc)
        torch.cuda.synchronize()
        assert np.array_equal(ok.cpu().numpy(), want)
    ks.close()
    ctx.close()
