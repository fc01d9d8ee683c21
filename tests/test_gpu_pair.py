"""The two-block kernel of the 24-field system on both sides of the size from which it writes non-temporally (a step: 800
blocks; an evaluation: 813), with single blocks and all sorts of neighbours; against the oracle, which runs the same sequence."""
import numpy as np
import pytest
import torch

import paper_2007_12792_amd as octfd
import synthdata as sd
from helpers import assert_close, dev_empty

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("radius,stream", [(0.01, False), (0.06, True)])
def test_evaluation_and_step(orc, dev, radius, stream):
    p = dict(lmin=3, lmax=5, pts_q20=sd.seed_points("rand", 1), radius_q20=np.full(2, int(radius * sd.Q), np.uint32))
    to, tg = orc.Tree.build(**p), octfd.Tree.build(**p)
    print(tg.n, flush=True)
    assert (48 * 4096 * tg.n > 160000000) == stream and (96 * 4096 * tg.n > 300 << 20) == stream
    u = sd.make_fields("C4", to.leaves).numpy()
    ud = torch.from_numpy(u).to(dev)
    out = dev_empty(u.shape, dev)
    tg.rhs_eval_zipped(octfd.SYN24, ud, out, sigma=0.3)
    assert_close(out.cpu().numpy(), to.F(orc.SYN24, u, sigma=0.3), "evaluation, %d blocks" % tg.n)
    ws = torch.empty(tg.rk_workspace_bytes(octfd.SYN24) // 8, dtype=torch.float64, device=dev)
    tg.rk_step(octfd.SYN24, ud, 1e-6, ws, sigma=0.3)
    assert_close(ud.cpu().numpy(), to.rk4_step(orc.SYN24, u, 1e-6, sigma=0.3), "step, %d blocks" % tg.n)
