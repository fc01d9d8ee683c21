"""The fills of the virtual blocks with every number of variables at which they share a workgroup differently (1..7: a
wavefront takes one variable of one of several virtual blocks; 8: one each; more: several), against the oracle; and the
property of balanced trees that lets the centred fill run in one launch."""
import numpy as np
import pytest
import torch

import paper_2007_12792_amd as octfd
import synthdata as sd
from helpers import assert_close, dev_empty


@pytest.mark.gpu
@pytest.mark.parametrize("centred", [False, True])
@pytest.mark.parametrize("nvar", [1, 2, 3, 4, 5, 7, 8, 9, 17])
def test_unzip_with_any_number_of_variables(orc, dev, nvar, centred):
    # an uneven number of virtual blocks, so that the last workgroup is partly filled
    p = dict(lmin=3, lmax=5, pts_q20=np.array([[500000, 520000, 540000]], np.uint32), radius_q20=np.array([60000, 40000], np.uint32))
    to, tg = orc.Tree.build(**p), octfd.Tree.build(**p)
    u = np.random.default_rng(nvar).standard_normal((nvar, to.n, 8, 8, 8))
    got = dev_empty((nvar, tg.n, 14, 14, 14), dev)
    (tg.unzip_centred if centred else tg.unzip)(torch.from_numpy(u).to(dev), got)
    torch.cuda.synchronize()
    assert_close(got.cpu().numpy(), to.unzip_centred(u) if centred else to.unzip(u), "%d variables" % nvar)


@pytest.mark.parametrize("seed", range(6))
def test_centred_fill_reads_no_coarser_leaf(seed):
    """A needed child octant of a leaf L has no neighbour of L coarser than L on its own side."""
    rng = np.random.default_rng(seed)
    lmax = 5 + seed % 3
    t = octfd.Tree.build(3, lmax, rng.integers(0, 1 << 20, (1 + seed % 3, 3)).astype(np.uint32),
                         rng.integers(1, 60000, lmax - 3).astype(np.uint32))
    g, lv = t.ghost_table(), t.leaves.astype(np.int64)
    d = np.arange(27)
    step = np.stack([d % 3 - 1, d // 3 % 3 - 1, d // 9 - 1], axis=1)
    b, dirs = np.nonzero(g[:, :, 0] == 2)
    low = (lv[b, 1:] + step[dirs]) & 1                       # the octant: which half of its source leaf per axis
    src = g[b, dirs, 1]
    towards = 2 * low - 1
    assert len(b)
    for m in range(1, 8):
        s = towards * np.array([m & 1, m >> 1 & 1, m >> 2])
        assert (g[src, (s[:, 2] + 1) * 9 + (s[:, 1] + 1) * 3 + s[:, 0] + 1, 0] != 2).all()
