"""Sign of the host pipeline runs in the form that a persistent context chooses by itself: for every chunk it
evaluates the same number of candidates."""
import numpy as np
import pytest

from paper_2211_12265_amd import workload

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("level,chunk", [(2, 300), (87, 40)])
def test_chunks_run_in_the_automatic_form(level, chunk):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_12265_amd import dilithium as dl
    from paper_2211_12265_amd.pipeline import HostPipeline, pinned
    n = 2 * chunk
    pkl, skl, sgl = dl.sizes(level)
    ctx = dl.Context(0, mode=dl.MODE_PERSISTENT)
    pk, sk = (torch.zeros((n, w), dtype=torch.uint8, device="cuda") for w in (pkl, skl))
    ctx.keygen(level, torch.from_numpy(workload.keygen_seeds(n, seed=150)).cuda(), pk, sk)
    msg, off = workload.messages(workload.fixed_lengths(n, 32), seed=150)
    h_sk, h_msg, h_sig = pinned((n, skl)), pinned((len(msg),)), pinned((n, sgl))
    h_sk.copy_(sk)
    h_msg.numpy()[:] = msg
    p = HostPipeline(level, n_streams=2, chunk=chunk)
    p.sign(h_sk, h_msg, off, h_sig)
    torch.cuda.synchronize()
    gm = torch.from_numpy(msg).cuda()
    for s in range(2):
        a, b = s * chunk, (s + 1) * chunk
        sig = torch.zeros((chunk, sgl), dtype=torch.uint8, device="cuda")
        ctx.sign(level, sk[a:b], gm, torch.from_numpy(off[a:b + 1].astype(np.int64)).cuda(), sig)
        assert p.ctx[s].sign_stats() == ctx.sign_stats()
        assert np.array_equal(sig.cpu().numpy(), h_sig.numpy()[a:b])
    p.close()
    ctx.close()
