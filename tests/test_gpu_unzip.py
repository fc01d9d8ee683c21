"""unzip where its workgroups share the work differently: one per block for all variables (many blocks, or fewer than four
variables) or several (small trees), and an output that starts 8 bytes off a 16-byte boundary; against the oracle."""
import numpy as np
import pytest
import torch

import paper_2007_12792_amd as octfd
from helpers import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lmin,lmax,radius,nvar", [(3, 3, [], 1), (3, 3, [], 24), (3, 5, [50000, 30000], 5), (4, 4, [], 3), (4, 5, [50000], 5)])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("centred", [False, True])
def test_unzip(orc, dev, lmin, lmax, radius, nvar, shift, centred):
    p = dict(lmin=lmin, lmax=lmax, pts_q20=np.array([[500000, 300000, 1040000]], np.uint32), radius_q20=np.array(radius, np.uint32))
    to, tg = orc.Tree.build(**p), octfd.Tree.build(**p)
    u = np.random.default_rng(nvar).standard_normal((nvar, to.n, 8, 8, 8))
    # values outside the array must stay: one in front with the shift, and one behind
    buf = torch.full((shift + nvar * tg.n * 14 ** 3 + 1,), float("nan"), dtype=torch.float64, device=dev)
    got = buf[shift:-1].view(nvar, tg.n, 14, 14, 14)
    (tg.unzip_centred if centred else tg.unzip)(torch.from_numpy(u).to(dev), got)
    torch.cuda.synchronize()
    print(tg.n, nvar, shift, centred, flush=True)
    assert_close(got.cpu().numpy(), to.unzip_centred(u) if centred else to.unzip(u), "%d blocks, %d variables" % (tg.n, nvar))
    assert torch.isnan(buf[-1]) and (not shift or torch.isnan(buf[0]))
