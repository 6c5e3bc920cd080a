"""Secret keys whose s2 rows encode -5 (eta = 2) or -11 (eta = 4) in every coefficient, beyond what KeyGen
makes, signed by every form against the oracle.  c s2 then reaches past beta, and in each of these tasks
the sequential algorithm's signature has a low part of w that c s2 moves into the next interval (found by
signing message after message on the CPU, once with LowBits(w - c s2) and once with LowBits(w) - c s2)."""
import numpy as np
import pytest

import oracle
from paper_2211_12265_amd import workload

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPE = {2: (4, 4, 96), 3: (6, 5, 128), 5: (8, 7, 96)}   # k, l, bytes of a packed s poly
SEED = {2: 700, 3: 701, 5: 702}
# little-endian 4-byte messages
TASKS = {2: [5460, 6362, 8302, 8474, 8618, 14491, 14595, 17519, 20332, 22187, 22723, 23627, 24323, 24486, 24584,
             24800, 26610, 32765, 36577, 37295, 37852],
         3: [1050, 1918, 2022, 3337, 3700, 3822, 10060, 12553, 12579, 12839, 15025, 15800, 16515, 18665],
         5: [18242, 47572, 57878]}


@pytest.mark.parametrize("form", ["staged", "rounds", "few", "loop", "table"])
@pytest.mark.parametrize("level", [2, 3, 5])
def test_s2_beyond_eta(level, form):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_12265_amd import dilithium as dl
    k, l, eb = SHAPE[level]
    _, sk = oracle.keygen_batch(level, workload.keygen_seeds(1, seed=SEED[level]))
    sk = sk.copy()
    sk[:, 96 + l * eb:96 + (l + k) * eb] = 0xFF
    who = TASKS[level][:8] if form == "few" else (9 * TASKS[level])[:max(9, len(TASKS[level]))]
    n = len(who)
    msg = np.array(who, dtype="<u4").view(np.uint8)
    off = 4 * np.arange(n + 1, dtype=np.uint64)
    zero = np.zeros(n, dtype=np.uint32)
    want, _ = oracle.sign_batch(level, sk, msg, off, key_idx=zero)
    ctx = dl.Context(0, mode=dl.MODE_STAGED if form == "staged" else dl.MODE_PERSISTENT)
    if form == "loop":
        ctx.set_param("persist.hmax", 4)
    sig = torch.zeros(want.shape, dtype=torch.uint8, device="cuda")
    args = torch.from_numpy(msg).cuda(), torch.from_numpy(off.astype(np.int64)).cuda(), sig
    idx = torch.from_numpy(zero.astype(np.int32)).cuda()
    if form == "table":
        ks = dl.KeySet(ctx, level, sk=torch.from_numpy(sk).cuda())
        ks.sign(ctx, idx, *args)
    else:
        ctx.sign(level, torch.from_numpy(sk).cuda(), *args, key_idx=idx)
    torch.cuda.synchronize()
    assert np.array_equal(sig.cpu().numpy(), want)
    ctx.close()
