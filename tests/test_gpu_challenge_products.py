"""The challenge products on the matrix cores (c s1, c s2, c t0 as int8 tiles) at the edges of their
operands: secret keys whose t0 rows start with both extremes of the 13-bit range (4096 and -4095, the ends
of its two int8 parts) and whose s rows start with +-eta, signed against the oracle.  Levels 2 / 3 / 5 have
one full tile, a part-filled second one and two full ones."""
import numpy as np
import pytest

import oracle
from paper_2211_12265_amd import workload

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPE = {2: (4, 4, 96, 96), 3: (6, 5, 128, 96), 5: (8, 7, 96, 96)}   # k, l, bytes of a packed s poly, offset of s1


@pytest.mark.parametrize("mode", ["staged", "persistent"])
@pytest.mark.parametrize("level", [2, 3, 5])
def test_extreme_secrets(level, mode):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_12265_amd import dilithium as dl
    k, l, eb, off_s = SHAPE[level]
    n = 24
    _, sk = oracle.keygen_batch(level, workload.keygen_seeds(n, seed=600 + level))
    sk = sk.copy()
    top = {2: 4, 3: 8, 5: 4}[level] * (0x249249 if eb == 96 else 0x11111111)   # eta - v with v = 2 eta: -eta
    for t in range(n):
        for p in range(k + l):   # one word of coefficients eta (v = 0), one of -eta
            o = off_s + p * eb
            sk[t, o:o + 3] = 0
            sk[t, o + 3:o + 6] = np.frombuffer(np.uint32(top & 0xFFFFFF).tobytes()[:3], dtype=np.uint8)
        for p in range(k):       # eight coefficients 4096 (v = 0), eight of -4095 (v = 8191)
            o = off_s + (k + l) * eb + p * 416
            sk[t, o:o + 13] = 0x00
            sk[t, o + 13:o + 26] = 0xFF
    msg, off = workload.messages(workload.uniform_lengths(n, 0, 80, seed=level), seed=level)
    osig, _ = oracle.sign_batch(level, sk, msg, off)
    ctx = dl.Context(0, mode=dl.MODE_STAGED if mode == "staged" else dl.MODE_PERSISTENT)
    sig = torch.zeros(osig.shape, dtype=torch.uint8, device="cuda")
    ctx.sign(level, torch.from_numpy(sk).cuda(), torch.from_numpy(msg).cuda(),
             torch.from_numpy(off.astype(np.int64)).cuda(), sig)
    torch.cuda.synchronize()
    assert np.array_equal(sig.cpu().numpy(), osig)
    ctx.close()
