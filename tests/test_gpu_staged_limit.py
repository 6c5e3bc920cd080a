"""The staged form gives a task 4,096 loop rounds, whether a launch takes one nonce of many tasks or up to 64
nonces of few: a key whose t0 lets one nonce in some 5,000 pass, messages that need 4,048 and 4,068 nonces,
which are signed as the oracle does, and one that needs 4,101, which is refused."""
import numpy as np
import pytest

import oracle
from paper_2211_12265_amd import workload

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

T0, T0_BYTES = 864, 4 * 416


@pytest.mark.parametrize("others", [0, 600])   # tasks of an ordinary key: rounds of all before rounds of few
@pytest.mark.parametrize("message,nonces", [(532, 4048), (428, 4068), (222, 4101)])
def test_rounds_per_task(message, nonces, others):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_12265_amd import dilithium as dl
    _, sk = oracle.keygen_batch(2, workload.keygen_seeds(2, seed=900))
    sk = sk.copy()
    ext = np.repeat(np.random.default_rng(900).integers(0, 2, size=(1, 4, 256, 1), dtype=np.uint8), 13, axis=3)
    sk[0, T0:T0 + T0_BYTES] = np.packbits(ext.reshape(1, -1), axis=1, bitorder="little")
    idx = np.array([0] + [1] * others, dtype=np.uint32)
    msg = np.array([message] + list(range(others)), dtype="<u4").view(np.uint8)
    off = 4 * np.arange(idx.size + 1, dtype=np.uint64)
    ctx = dl.Context(0)
    sig = torch.zeros((idx.size, dl.sizes(2)[2]), dtype=torch.uint8, device="cuda")

    def call():
        ctx.sign(2, torch.from_numpy(sk).cuda(), torch.from_numpy(msg).cuda(),
                 torch.from_numpy(off.astype(np.int64)).cuda(), sig, key_idx=torch.from_numpy(idx.astype(np.int32)).cuda())
        torch.cuda.synchronize()
    if nonces > 4096:
        with pytest.raises(dl.DilError, match="did not terminate"):
            call()
    else:
        call()
        want, iters = oracle.sign_batch(2, sk, msg, off, key_idx=idx)
        assert iters[0] == nonces
        assert np.array_equal(sig.cpu().numpy(), want)
        assert ctx.sign_stats() == (int(iters.sum()), int(iters.sum()))
    ctx.close()
