"""The slab kernels of the kinds with one or two variables where they can go wrong: all three sorts of neighbours beyond every
face (one and two centres, the periodic corner), a uniform tree, and sizes on both sides of the one from which they run with
non-temporal accesses; against the oracle, which runs the same IEEE sequence."""
import numpy as np
import pytest
import torch

import paper_2007_12792_amd as octfd
import synthdata as sd
from helpers import KIND, assert_close, dev_empty

pytestmark = pytest.mark.gpu

TREES = {
    "uniform": dict(lmin=3, lmax=3, pts_q20=np.zeros((0, 3), np.uint32), radius_q20=np.zeros(0, np.uint32)),
    "corner": dict(lmin=3, lmax=5, pts_q20=np.array([[1000, 2000, 1040000]], np.uint32), radius_q20=np.array([50000, 60000], np.uint32)),
    "two": dict(lmin=3, lmax=6, pts_q20=np.array([[400000, 300000, 600000], [700000, 650000, 500000]], np.uint32),
                radius_q20=np.array([30000, 20000, 9000], np.uint32)),
}


@pytest.mark.parametrize("tree", sorted(TREES))
@pytest.mark.parametrize("kind", ["DERIVS", "WAVE", "BURGERS"])
def test_evaluation_and_step(orc, dev, kind, tree):
    to, tg = orc.Tree.build(**TREES[tree]), octfd.Tree.build(**TREES[tree])
    k = KIND[kind]
    u = np.random.default_rng(3).standard_normal((octfd.nvar_in(k), to.n, 8, 8, 8))
    ud = torch.from_numpy(u).to(dev)
    out = dev_empty((octfd.nvar_out(k), tg.n, 8, 8, 8), dev)
    tg.rhs_eval_zipped(k, ud, out, sigma=0.3)
    assert_close(out.cpu().numpy(), to.F(k, u, sigma=0.3), "%s %s" % (kind, tree))
    if octfd.nvar_in(k) == octfd.nvar_out(k):
        ws = torch.empty(tg.rk_workspace_bytes(k) // 8, dtype=torch.float64, device=dev)
        tg.rk_step(k, ud, 1e-4, ws, sigma=0.3)
        assert_close(ud.cpu().numpy(), to.rk4_step(k, u, 1e-4, sigma=0.3), "step %s %s" % (kind, tree))


@pytest.mark.parametrize("kind,radius,stream", [("DERIVS", 0.1105, False), ("DERIVS", 0.1115, True), ("WAVE", 0.122, False), ("WAVE", 0.13, True),
                                                ("BURGERS", 0.16, False), ("BURGERS", 0.18, True)])
def test_both_sides_of_the_streaming_size(orc, dev, kind, radius, stream):
    """DERIVS on 7,750 and 7,904 blocks (159 and 162 MB in and out); WAVE on 9,570 and 10,830 (a step's vectors: 314 and
    355 MB); Burgers on 17,018 and 22,478 blocks (279 and 368 MB)."""
    p = dict(lmin=3, lmax=6, pts_q20=sd.seed_points("rand", 1), radius_q20=np.full(3, int(radius * sd.Q), np.uint32))
    to, tg = orc.Tree.build(**p), octfd.Tree.build(**p)
    print(kind, tg.n, flush=True)
    k = KIND[kind]
    vectors = octfd.nvar_in(k) + octfd.nvar_out(k) if kind == "DERIVS" else 4 * octfd.nvar_in(k)
    assert (vectors * 4096 * tg.n > (160000000 if kind == "DERIVS" else 300 << 20)) == stream
    u = np.random.default_rng(5).standard_normal((octfd.nvar_in(k), to.n, 8, 8, 8))
    ud = torch.from_numpy(u).to(dev)
    if kind == "DERIVS":
        out = dev_empty((4, tg.n, 8, 8, 8), dev)
        tg.rhs_eval_zipped(k, ud, out)
        assert_close(out.cpu().numpy(), to.F(k, u), "%s %d blocks" % (kind, tg.n))
    else:
        ws = torch.empty(tg.rk_workspace_bytes(k) // 8, dtype=torch.float64, device=dev)
        tg.rk_step(k, ud, 1e-5, ws, sigma=0.3)
        assert_close(ud.cpu().numpy(), to.rk4_step(k, u, 1e-5, sigma=0.3), "step %s %d blocks" % (kind, tg.n))
