"""KeyGen's secrets are picked out of the squeezed streams by the kernel that needs them: seeds whose
streams hold fewer than 256 accepted nibbles in their first two blocks (found by search; polynomial and
count beside each), where a third one is squeezed and read, and eta = 2, where they never do."""
import hashlib
import struct

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (seed number, polynomial, accepted nibbles of the first 272 bytes)
SHORT = {3: [(14857, 1, 252), (25783, 6, 255)], 65: [(10063, 9, 248), (14708, 6, 255)]}


@pytest.mark.parametrize("level", [2, 3, 65, 87])
def test_short_streams(level):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_12265_amd import dilithium as dl
    numbers = [i for i, _, _ in SHORT.get(level, [])] + list(range(60))
    seeds = np.stack([np.frombuffer(struct.pack("<Q", i) + bytes(24), dtype=np.uint8) for i in numbers])
    for (_, r, want), seed in zip(SHORT.get(level, []), seeds):
        rhop = hashlib.shake_256(seed.tobytes() + (b"\x06\x05" if level == 65 else b"")).digest(96)[32:]
        stream = np.frombuffer(hashlib.shake_256(rhop + struct.pack("<H", r)).digest(272), dtype=np.uint8)
        assert int(((stream & 15) < 9).sum() + ((stream >> 4) < 9).sum()) == want < 256
    opk, osk = oracle.keygen_batch(level, seeds)
    pk = torch.zeros(opk.shape, dtype=torch.uint8, device="cuda")
    sk = torch.zeros(osk.shape, dtype=torch.uint8, device="cuda")
    ctx = dl.Context(0)
    ctx.keygen(level, torch.from_numpy(seeds).cuda(), pk, sk)
    torch.cuda.synchronize()
    assert np.array_equal(pk.cpu().numpy(), opk) and np.array_equal(sk.cpu().numpy(), osk)
    ctx.close()
