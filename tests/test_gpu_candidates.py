"""A workgroup per candidate: rounds of up to 8 tasks and one more, and the staged form's loop over the tasks
that are few enough (2048 mask streams) for a workgroup each, also with keys whose t0 makes most
candidates fail, so that tasks need more than the 64 nonces of one launch.  Everything equals the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2211_12265_amd import workload

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _check(level, sk, n, mode, extra=None):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_12265_amd import dilithium as dl
    msg, off = workload.messages(workload.uniform_lengths(n, 0, 300, seed=n + level), seed=n)
    want, iters = oracle.sign_batch(level, sk, msg, off)
    if extra:
        extra(iters)
    ctx = dl.Context(0, mode=dl.MODE_STAGED if mode == "staged" else dl.MODE_PERSISTENT)
    sig = torch.zeros(want.shape, dtype=torch.uint8, device="cuda")
    ctx.sign(level, torch.from_numpy(sk).cuda(), torch.from_numpy(msg).cuda(),
             torch.from_numpy(off.astype(np.int64)).cuda(), sig)
    torch.cuda.synchronize()
    assert np.array_equal(sig.cpu().numpy(), want)
    evaluated, sequential = ctx.sign_stats()
    assert sequential == int(iters.sum())
    assert evaluated == sequential if mode == "staged" else evaluated >= sequential
    ctx.close()


@pytest.mark.parametrize("level", [2, 3, 5, 44, 65, 87])
@pytest.mark.parametrize("mode,count", [("persistent", 1), ("persistent", 8), ("persistent", 9), ("staged", 1)])
def test_few_tasks(level, mode, count):
    _, sk = oracle.keygen_batch(level, workload.keygen_seeds(count, seed=1000 + level))
    _check(level, sk, count, mode)


@pytest.mark.parametrize("level,count", [(44, 512), (44, 513), (3, 409), (3, 410), (87, 292), (87, 293)])
def test_staged_counts_where_the_loop_changes(level, count):
    _, sk = oracle.keygen_batch(level, workload.keygen_seeds(count, seed=1010 + level))
    _check(level, sk, count, "staged")


@pytest.mark.parametrize("mode", ["staged", "persistent"])
@pytest.mark.parametrize("level,frac", [(2, 0.6), (3, 0.8), (5, 0.7)])
def test_more_nonces_than_one_launch(level, frac, mode):
    n, (k, t0_off) = 48, {2: (4, 864), 3: (6, 1504), 5: (8, 1536)}[level]
    g = np.random.default_rng(1020 + level)
    _, sk = oracle.keygen_batch(level, workload.keygen_seeds(n, seed=1020 + level))
    sk = sk.copy()
    bits = np.unpackbits(sk[:, t0_off:t0_off + 416 * k], axis=1, bitorder="little").reshape(n, k, 256, 13)
    ext = g.random((n, k, 256)) < frac
    bits[ext] = g.integers(0, 2, size=int(ext.sum()), dtype=np.uint8)[:, None]
    sk[:, t0_off:t0_off + 416 * k] = np.packbits(bits.reshape(n, -1), axis=1, bitorder="little")
    msg, off = workload.messages(workload.uniform_lengths(8, 0, 300, seed=8 + level), seed=8)   # as in _check
    need = np.concatenate([oracle.sign_batch(level, sk[i:i + 8], msg, off)[1] for i in range(0, n, 8)])
    first = 8 * int(need.reshape(-1, 8).max(axis=1).argmax())

    def enough(iters):
        assert (iters > 64).any()
    _check(level, sk[first:first + 8], 8, mode, enough)
