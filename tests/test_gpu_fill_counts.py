"""The fills of the virtual blocks with every number of variables at which they share a workgroup differently (few: a
wavefront takes one variable of one of several virtual blocks; 8: one each; more: several), against the oracle; and the
properties of balanced trees that let the centred fill run in one launch and leave no workgroup of a fill partly filled."""
import numpy as np
import pytest
import torch

import paper_2007_12792_amd as octfd
from helpers import assert_close, dev_empty


def virtual_blocks(t):
    """how many: the distinct pairs of source leaf and child octant among the coarser entries of the ghost table"""
    g, lv, d = t.ghost_table(), t.leaves.astype(np.int64), np.arange(27)
    b, dirs = np.nonzero(g[:, :, 0] == 2)
    low = (lv[b, 1:] + np.stack([d % 3 - 1, d // 3 % 3 - 1, d // 9 - 1], axis=1)[dirs]) & 1
    return np.unique(g[b, dirs, 1].astype(np.int64) * 8 + low @ np.array([1, 2, 4])).size


@pytest.mark.parametrize("seed", range(6))
def test_virtual_blocks_come_in_eights(seed):
    """A child octant of a leaf L lies at a corner of L, and is needed if one of the seven octants around that corner is
    subdivided.  Balance makes all eight octants around such a corner exist, so with s of them subdivided it has 8 - s virtual
    blocks; every subdivided octant is counted at its eight corners: 8 * corners - 8 * subdivided octants.  A workgroup of a
    fill takes 1, 2, 4 or 8 virtual blocks, so none is partly filled."""
    rng = np.random.default_rng(seed)
    base = octfd.Tree.build(3, 3, np.zeros((0, 3), np.uint32), np.zeros(0, np.uint32)).leaves
    pick = rng.choice(512, rng.integers(1, 200), replace=False)
    kids = [np.stack([np.full(pick.size, 4), 2 * base[pick, 1] + (c & 1), 2 * base[pick, 2] + (c >> 1 & 1), 2 * base[pick, 3] + (c >> 2)], 1) for c in range(8)]
    n = virtual_blocks(octfd.Tree.from_leaves(np.concatenate([np.delete(base, pick, 0), *kids])))
    assert n and n % 8 == 0
    deep = octfd.Tree.build(3, 6, rng.integers(0, 1 << 20, (1 + seed % 3, 3)).astype(np.uint32), rng.integers(1, 80000, 3).astype(np.uint32))
    assert virtual_blocks(deep) and virtual_blocks(deep) % 8 == 0


@pytest.mark.gpu
@pytest.mark.parametrize("centred", [False, True])
@pytest.mark.parametrize("nvar", [1, 2, 3, 4, 5, 7, 8, 9, 17])
def test_unzip_with_any_number_of_variables(orc, dev, nvar, centred):
    # 304 virtual blocks: with every number of variables the grid, a multiple of 128, has workgroups beyond the last virtual
    # block; with 3, 5 and 7 variables wavefronts of every workgroup have none
    p = dict(lmin=3, lmax=5, pts_q20=np.array([[500000, 520000, 540000]], np.uint32), radius_q20=np.array([60000, 40000], np.uint32))
    to, tg = orc.Tree.build(**p), octfd.Tree.build(**p)
    assert virtual_blocks(tg) == 304 and 304 // (8 // min(nvar, 8)) % 128
    u = np.random.default_rng(nvar).standard_normal((nvar, to.n, 8, 8, 8))
    got = dev_empty((nvar, tg.n, 14, 14, 14), dev)
    (tg.unzip_centred if centred else tg.unzip)(torch.from_numpy(u).to(dev), got)
    torch.cuda.synchronize()
    assert_close(got.cpu().numpy(), to.unzip_centred(u) if centred else to.unzip(u), "%d variables" % nvar)


@pytest.mark.gpu
@pytest.mark.parametrize("nvar", [1, 2, 3, 4])
@pytest.mark.parametrize("radii,virtual", [([60000, 40000, 0], 304), ([170000, 105000, 60000], 1488), ([110000, 60000, 40000], 2064), ([200000, 130000, 80000], 3888)])
def test_centred_fill_with_every_number_of_virtual_blocks_per_workgroup(orc, dev, nvar, radii, virtual):
    """One variable: 1, 2, 4 and 8 virtual blocks per workgroup (halved while 768 workgroups hold them all); two: 1, 2, 4 and 4."""
    pts = np.array([[500000, 520000, 540000]] if virtual < 2000 else [[300000, 520000, 540000], [800000, 100000, 200000]], np.uint32)
    p = dict(lmin=3, lmax=5 if virtual == 304 else 6, pts_q20=pts, radius_q20=np.array(radii, np.uint32))
    to, tg = orc.Tree.build(**p), octfd.Tree.build(**p)
    assert virtual_blocks(tg) == virtual
    u = np.random.default_rng(nvar).standard_normal((nvar, to.n, 8, 8, 8))
    got = dev_empty((nvar, tg.n, 14, 14, 14), dev)
    tg.unzip_centred(torch.from_numpy(u).to(dev), got)
    torch.cuda.synchronize()
    assert_close(got.cpu().numpy(), to.unzip_centred(u), "%d variables, %d virtual blocks" % (nvar, virtual))


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
