"""The 24-field kernel on padded blocks against the oracle: same results to the bit, on trees of one round of 256 units, of a second that is
nearly empty and of several, with blocks without a partner.  Corners are never read, ghosts of the output never written, and padded
arrays may start at any double."""
import numpy as np
import pytest
import torch

import paper_2007_12792_amd as octfd
import synthdata as sd

from test_gpu_brick import shifted

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lmax,style,radius,ratio", [(3, "rand", 0.0, 1.0), (4, "rand", 0.02, 1.0), (4, "rand", 0.12, 1.0), (5, "orbit", 0.083, 0.643),
                                                     (6, "rand", 0.05, 0.6)])
@pytest.mark.parametrize("by", [0, 1])
def test_padded_same_bits_as_the_oracle(orc, dev, lmax, style, radius, ratio, by):
    p = dict(lmin=3, lmax=lmax, pts_q20=sd.seed_points(style, 1), radius_q20=np.array([int(radius * ratio ** k * sd.Q) for k in range(lmax - 3)], dtype=np.uint32))
    t = octfd.Tree.build(**p)
    u = sd.make_fields("C4", t.leaves, 3, device="cuda")
    want = orc.Tree.build(**p).F(orc.SYN24, u.cpu().numpy(), sigma=0.3)
    print(t.n, "blocks, aligned to", 16 if by == 0 else 8, flush=True)
    padded = shifted(torch.zeros((24, t.n, 14, 14, 14), dtype=torch.float64, device=dev), by)
    t.unzip(u, padded)
    ghost = [slice(0, 3), slice(11, 14)]
    for z in ghost:
        for y in ghost:
            for x in ghost:
                padded[:, :, z, y, x] = float("nan")
    out = shifted(torch.full_like(padded, -7.5), by)
    t.rhs_eval(octfd.SYN24, padded, out, sigma=0.3)
    inner = out[:, :, 3:11, 3:11, 3:11]
    assert np.isfinite(want).all() and np.array_equal(inner.cpu().numpy(), want)
    inner.fill_(-7.5)
    assert (out == -7.5).all()
