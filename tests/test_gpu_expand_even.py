"""Sign in rounds at the counts where its ExpandA launch changes its workgroups (more than 131,072 and at
most 327,680 polynomials take 256 lanes), with partly filled last workgroups.  Equal to the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2211_12265_amd import workload

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("level,count", [(5, 2340), (87, 2341), (3, 4370), (5, 5851), (5, 5852)])
def test_counts_where_workgroups_change(level, count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_12265_amd import dilithium as dl
    nk = 41
    _, sk = oracle.keygen_batch(level, workload.keygen_seeds(nk, seed=1200 + level))
    key_idx = (np.arange(count) * 11 % nk).astype(np.uint32)
    msg, off = workload.messages(workload.fixed_lengths(count, 32), seed=count)
    want, _ = oracle.sign_batch(level, sk, msg, off, key_idx=key_idx)
    ctx = dl.Context(0, mode=dl.MODE_PERSISTENT)
    sig = torch.zeros(want.shape, dtype=torch.uint8, device="cuda")
    ctx.sign(level, torch.from_numpy(sk).cuda(), torch.from_numpy(msg).cuda(),
             torch.from_numpy(off.astype(np.int64)).cuda(), sig,
             key_idx=torch.from_numpy(key_idx.astype(np.int32)).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(sig.cpu().numpy(), want)
    ctx.close()
