"""The finishing launch of Sign in rounds with work to do: keys whose t0 makes most candidates fail leave many
tasks after the last round, fewer than its workgroups, about as many, and more, and in both groups of a call.
Signatures and statistics equal the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2211_12265_amd import workload

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

T0 = {2: (4, 864), 3: (6, 1504), 5: (8, 1536)}   # k, offset of t0 in the secret key


@pytest.mark.parametrize("level,frac,count", [(2, 0.6, 16), (2, 0.6, 700), (3, 1.0, 512), (5, 0.8, 40), (2, 0.5, 2600),
                                              (2, 0.5, 16385)])   # two groups
def test_tasks_left_after_the_rounds(level, frac, count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_12265_amd import dilithium as dl
    k, t0 = T0[level]
    g = np.random.default_rng(1100 + level)
    _, sk = oracle.keygen_batch(level, workload.keygen_seeds(count, seed=1100 + level))
    sk = sk.copy()
    bits = np.unpackbits(sk[:, t0:t0 + 416 * k], axis=1, bitorder="little").reshape(count, k, 256, 13)
    ext = g.random((count, k, 256)) < frac
    bits[ext] = g.integers(0, 2, size=int(ext.sum()), dtype=np.uint8)[:, None]
    sk[:, t0:t0 + 416 * k] = np.packbits(bits.reshape(count, -1), axis=1, bitorder="little")
    msg, off = workload.messages(workload.uniform_lengths(count, 0, 300, seed=level), seed=1100)
    want, iters = oracle.sign_batch(level, sk, msg, off)
    assert iters.mean() > 20
    ctx = dl.Context(0, mode=dl.MODE_PERSISTENT)
    sig = torch.zeros(want.shape, dtype=torch.uint8, device="cuda")
    ctx.sign(level, torch.from_numpy(sk).cuda(), torch.from_numpy(msg).cuda(),
             torch.from_numpy(off.astype(np.int64)).cuda(), sig)
    ctx.check()
    assert np.array_equal(sig.cpu().numpy(), want)
    evaluated, sequential = ctx.sign_stats()
    assert sequential == int(iters.sum()) and evaluated >= sequential
    ctx.close()
