"""The 24-field kernel with two points per thread, on arrays aligned to 16 bytes and to 8 bytes only, against the oracle.  Both run the same
sequence up to factors that are powers of two, so results are the same to the bit.  Trees of one round of 256 units, of a second that is nearly empty,
and of several, on both sides of the sizes for non-temporal accesses; with blocks without a partner next to finer, coarser and equal
neighbours."""
import numpy as np
import pytest
import torch

import paper_2007_12792_amd as octfd
import synthdata as sd

pytestmark = pytest.mark.gpu


def shifted(t, by):
    """a copy of t that starts 8 * by bytes into an allocation"""
    flat = torch.full((t.numel() + 2,), float("nan"), dtype=torch.float64, device=t.device)
    v = flat[by:by + t.numel()].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 16 == 8 * (by % 2)
    return v


@pytest.mark.parametrize("lmax,style,radius,ratio", [(3, "rand", 0.0, 1.0), (4, "rand", 0.02, 1.0), (4, "rand", 0.12, 1.0), (5, "orbit", 0.083, 0.643),
                                                     (6, "rand", 0.05, 0.6)])
def test_same_bits_as_the_oracle(orc, dev, lmax, style, radius, ratio):
    p = dict(lmin=3, lmax=lmax, pts_q20=sd.seed_points(style, 1), radius_q20=np.array([int(radius * ratio ** k * sd.Q) for k in range(lmax - 3)], dtype=np.uint32))
    to, t = orc.Tree.build(**p), octfd.Tree.build(**p)
    u = sd.make_fields("C4", t.leaves, 3, device="cuda")
    uh = u.cpu().numpy()
    want = [to.F(orc.SYN24, uh, sigma=0.3), to.rk4_step(orc.SYN24, uh, 1e-6, sigma=0.3), to.rk4_step_centred(orc.SYN24, uh, 1e-6, sigma=0.3)]
    t.upload()
    ws = torch.empty(t.rk_workspace_bytes(octfd.SYN24) // 8, dtype=torch.float64, device=dev)
    for by in (0, 1):
        print(t.n, "blocks, aligned to", 16 if by == 0 else 8, flush=True)
        v, out = shifted(u, by), shifted(torch.zeros_like(u), by)
        t.rhs_eval_zipped(octfd.SYN24, v, out, sigma=0.3)
        s, c = shifted(u, by), shifted(u, by)
        t.rk_step(octfd.SYN24, s, 1e-6, ws, sigma=0.3)
        t.rk_step_centred(octfd.SYN24, c, 1e-6, ws, sigma=0.3)
        for what, got, w in zip(("evaluation", "step", "centred step"), (out, s, c), want):
            got = got.cpu().numpy()
            assert np.isfinite(w).all() and np.array_equal(got, w), (what, by, int((got != w).sum()))
