"""Sign in rounds (the automatic form of the persistent mode) at the sizes where its launches change shape:
one task, the counts at which the masks and challenges go from 16-lane rows to lane pairs to single lanes
and the checks from a workgroup to a wavefront per task, and a second group; and with keys whose t0 makes
most candidates fail, so that tasks are left over for the finishing launch.  Every signature equals the
oracle's."""
import numpy as np
import pytest

import oracle
from paper_2211_12265_amd import workload

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _sign(level, sk, msg, off, key_idx=None):
    from paper_2211_12265_amd import dilithium as dl
    n = off.size - 1
    ctx = dl.Context(0, mode=dl.MODE_PERSISTENT)
    sig = torch.zeros((n, dl.sizes(level)[2]), dtype=torch.uint8, device="cuda")
    ctx.sign(level, torch.from_numpy(sk).cuda(), torch.from_numpy(msg).cuda(),
             torch.from_numpy(off.astype(np.int64)).cuda(), sig,
             key_idx=None if key_idx is None else torch.from_numpy(key_idx.astype(np.int32)).cuda())
    torch.cuda.synchronize()
    stats = ctx.sign_stats()
    ctx.close()
    return sig.cpu().numpy(), stats


@pytest.mark.parametrize("level,count", [(2, 1), (3, 3), (5, 128), (65, 129), (2, 1366), (44, 2049), (87, 1170),
                                         (2, 4097), (3, 5001), (2, 16385)])
def test_counts_where_launches_change(level, count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nk = min(count, 37)
    _, sk = oracle.keygen_batch(level, workload.keygen_seeds(nk, seed=800 + level))
    key_idx = (np.arange(count) * 5 % nk).astype(np.uint32)
    msg, off = workload.messages(workload.uniform_lengths(count, 0, 200, seed=count), seed=count)
    want, iters = oracle.sign_batch(level, sk, msg, off, key_idx=key_idx)
    got, (evaluated, sequential) = _sign(level, sk, msg, off, key_idx)
    assert np.array_equal(got, want)
    assert sequential == int(iters.sum()) and evaluated >= sequential


@pytest.mark.parametrize("level,frac", [(2, 0.6), (3, 0.8), (5, 0.7)])
def test_tasks_left_after_the_rounds(level, frac):
    """A fraction of the t0 coefficients at the ends of their range: the hints overflow omega most of the
    time and several tasks need more nonces than all rounds together hand out (at most 64 here)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, (k, t0_off) = 24, {2: (4, 864), 3: (6, 1504), 5: (8, 1536)}[level]
    g = np.random.default_rng(700 + level)
    _, sk = oracle.keygen_batch(level, workload.keygen_seeds(n, seed=700 + level))
    sk = sk.copy()
    bits = np.unpackbits(sk[:, t0_off:t0_off + 416 * k], axis=1, bitorder="little").reshape(n, k, 256, 13)
    ext = g.random((n, k, 256)) < frac
    bits[ext] = g.integers(0, 2, size=int(ext.sum()), dtype=np.uint8)[:, None]
    sk[:, t0_off:t0_off + 416 * k] = np.packbits(bits.reshape(n, -1), axis=1, bitorder="little")
    msg, off = workload.messages(workload.fixed_lengths(n, 32), seed=level)
    want, iters = oracle.sign_batch(level, sk, msg, off)
    assert (iters > 64).sum() >= 2
    got, (_, sequential) = _sign(level, sk, msg, off)
    assert np.array_equal(got, want)
    assert sequential == int(iters.sum())
