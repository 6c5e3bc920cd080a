"""10,000 tasks in the form a persistent context chooses by itself (rounds), at every parameter set: all
signatures equal the oracle's, deterministic and randomized, launched directly and replayed from a graph with
eager work in between."""
import numpy as np
import pytest

import oracle
from paper_2211_12265_amd import workload

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("level,mix,hedged", [(2, "fixed32", False), (3, "uniform", True), (5, "uniform", False),
                                              (44, "fixed32", True), (65, "uniform", False), (87, "uniform", True)])
def test_ten_thousand_tasks_in_rounds(level, mix, hedged):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_12265_amd import dilithium as dl
    n = 10000
    pkl, skl, sgl = dl.sizes(level)
    ctx = dl.Context(0, mode=dl.MODE_PERSISTENT)
    pk, sk = (torch.zeros((n, w), dtype=torch.uint8, device="cuda") for w in (pkl, skl))
    ctx.keygen(level, torch.from_numpy(workload.keygen_seeds(n, seed=400 + level)).cuda(), pk, sk)
    lens = workload.fixed_lengths(n, 32) if mix == "fixed32" else workload.uniform_lengths(n, 32, 4096, seed=level)
    msg, off = workload.messages(lens, seed=400 + level)
    rnd = workload.random_bytes("test/rnd", 400 + level, (n, 32 if level in dl.MLDSA_LEVELS else 64)) if hedged else None
    want, iters = oracle.sign_batch(level, sk.cpu().numpy(), msg, off, rnd=rnd)
    gm, go = torch.from_numpy(msg).cuda(), torch.from_numpy(off.astype(np.int64)).cuda()
    gr = None if rnd is None else torch.from_numpy(rnd).cuda()
    sig = torch.empty((n, sgl), dtype=torch.uint8, device="cuda")
    ver = torch.zeros(n, dtype=torch.int32, device="cuda")
    for graph in (0, 1, 1, 1):   # direct, captured, replayed twice
        ctx.set_param("graph", graph)
        sig.zero_()
        ctx.sign(level, sk, gm, go, sig, rnd=gr)
        ctx.verify(level, pk, gm, go, sig, ver)
        assert int(ver.sum()) == n
        assert np.array_equal(sig.cpu().numpy(), want)
        assert ctx.sign_stats()[1] == int(iters.sum())
    ctx.check()
    ctx.close()
