"""The balance and the ghost table from neighbours of nodes with children, against the oracle's own walk: deep trees around the
periodic corner and edges, and leaf lists that break the balance across a face, an edge or a corner only."""
import time

import numpy as np
import pytest

import paper_2007_12792_amd as octfd
import synthdata as sd


def children(leaf):
    l, x, y, z = (int(v) for v in leaf)
    return np.array([[l + 1, 2 * x + (c & 1), 2 * y + (c >> 1 & 1), 2 * z + (c >> 2)] for c in range(8)], np.uint32)


@pytest.mark.parametrize("lmin,lmax,seed", [(3, 3, (0, 0, 0)), (3, 9, (0, 0, 0)), (3, 8, (1048575, 0, 524288)), (4, 9, (300001, 1048575, 7))])
def test_leaves_and_table(orc, lmin, lmax, seed):
    p = dict(lmin=lmin, lmax=lmax, pts_q20=np.array([seed], np.uint32), radius_q20=np.full(lmax - lmin, 3, np.uint32))
    to, tg = orc.Tree.build(**p), octfd.Tree.build(**p)
    assert (to.leaves == tg.leaves).all() and (to.ghost_table() == tg.ghost_table()).all()
    again = octfd.Tree.from_leaves(np.random.default_rng(1).permutation(tg.leaves))
    assert (again.ghost_table() == tg.ghost_table()).all()


@pytest.mark.parametrize("child,inner", [(0, 0), (0, 1), (7, 7), (7, 3), (2, 5)])
def test_unbalanced_leaf_lists_are_refused(child, inner):
    """A child of a level-3 leaf split once or twice more: its children touch level-3 leaves, two or three levels coarser."""
    base = octfd.Tree.build(3, 3, np.zeros((0, 3), np.uint32), np.zeros(0, np.uint32)).leaves
    kids = children(base[100])
    deep = children(kids[child])
    one = np.concatenate([np.delete(base, 100, 0), kids])
    assert octfd.Tree.from_leaves(one).n == 519
    two = np.concatenate([np.delete(base, 100, 0), np.delete(kids, child, 0), deep])
    with pytest.raises(octfd.OctfdError) as e:
        octfd.Tree.from_leaves(two)
    assert e.value.status == octfd.OT_E_UNBALANCED
    three = np.concatenate([np.delete(base, 100, 0), np.delete(kids, child, 0), np.delete(deep, inner, 0), children(deep[inner])])
    with pytest.raises(octfd.OctfdError) as e:
        octfd.Tree.from_leaves(three)
    assert e.value.status == octfd.OT_E_UNBALANCED


def test_handing_out_the_table_is_little_more_than_a_copy():
    """27,791 blocks: rows made one entry at a time take six copies of the table, as they are 1.4"""
    t = octfd.Tree.build(3, 8, sd.seed_points("orbit", 1), np.array([int(0.1 * 0.83 ** k * sd.Q) for k in range(5)], np.uint32))
    def fastest(go):
        times = []
        for _ in range(9):
            start = time.perf_counter()
            go()
            times.append(time.perf_counter() - start)
        return min(times)
    table = t.ghost_table()
    made, copied = fastest(t.ghost_table), fastest(table.copy)
    assert made < 3.5 * copied, (t.n, made, copied)
