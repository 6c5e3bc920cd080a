"""ExpandA and ExpandS on a wavefront per stream (at most 4096 polynomials beside
hash chains, 8192 streams alone) and KeyGen's seeds on the wide forms,
at the counts on both sides of the line, the smallest call, and seeds whose ExpandS streams need a third
block (found by search).  KeyGen, Sign and Verify equal the oracle; the last two expand A from their own rows."""
import struct

import numpy as np
import pytest

import oracle
from paper_2211_12265_amd import workload

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

THIRD_BLOCK = {3: [14857, 25783], 65: [10063, 14708]}


def _run(level, seeds):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_12265_amd import dilithium as dl
    n = len(seeds)
    pkl, skl, sgl = dl.sizes(level)
    opk, osk = oracle.keygen_batch(level, seeds)
    msg, off = workload.messages(workload.fixed_lengths(n, 33), seed=n)
    osig, _ = oracle.sign_batch(level, osk, msg, off)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    new = lambda w: torch.zeros((n, w), dtype=torch.uint8, device="cuda")
    ctx = dl.Context(0, mode=dl.MODE_PERSISTENT)
    pk, sk, sig = new(pkl), new(skl), new(sgl)
    ctx.keygen(level, dev(seeds), pk, sk)
    assert np.array_equal(pk.cpu().numpy(), opk) and np.array_equal(sk.cpu().numpy(), osk)
    dmsg, doff = dev(msg), dev(off.astype(np.int64))
    ctx.sign(level, sk, dmsg, doff, sig)
    ok = torch.full((n,), 9, dtype=torch.int32, device="cuda")
    ctx.verify(level, pk, dmsg, doff, sig, ok)
    torch.cuda.synchronize()
    assert np.array_equal(sig.cpu().numpy(), osig) and bool((ok == 1).all())
    ctx.close()


@pytest.mark.parametrize("level,count", [(2, 1), (65, 1), (87, 1), (2, 85), (44, 86), (44, 128), (2, 129), (3, 49),
                                         (65, 50), (3, 68), (65, 69), (5, 28), (87, 29), (87, 36), (5, 37),
                                         (2, 256), (44, 257), (3, 136), (65, 137), (2, 341), (44, 342), (3, 199),
                                         (65, 200), (5, 73), (87, 74), (5, 115), (87, 116)])
def test_counts_where_the_expansions_change(level, count):
    _run(level, workload.keygen_seeds(count, seed=1100 + level))


@pytest.mark.parametrize("level", [3, 65])
def test_third_block(level):
    _run(level, np.stack([np.frombuffer(struct.pack("<Q", i) + bytes(24), dtype=np.uint8)
                          for i in THIRD_BLOCK[level]]))


@pytest.mark.parametrize("count", [1, 3, 2048, 2049, 8192, 8193])
def test_expand_a_primitive(count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_12265_amd import dilithium as dl
    seeds = workload.random_bytes("test/expand_a_wave", count, (count, 34))
    want = oracle.expand_a_polys(seeds)
    out = torch.zeros((count, 256), dtype=torch.int32, device="cuda")
    ctx = dl.Context(0)
    ctx.expand_a(torch.from_numpy(seeds).cuda(), out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), want)
    ctx.close()
