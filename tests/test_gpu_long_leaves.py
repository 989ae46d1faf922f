"""Leaves of more particles than a walk group: runs of points in one cell of the
finest level (longest a few thousand), and large leaves whose boxes exceed the size
limit of groups. Nodes, moments and groups equal the CPU oracle's (the oracle's
order of FP64 operations and of particles). Points many times over, exactly or
nearly, are sorted in the stable order of their keys."""
import numpy as np
import pytest
import torch

import oracle
from paper_2110_11658_amd import ic

pytestmark = pytest.mark.gpu


def _points(kind):
    c = ic.plummer(3000, seed=41, masses="kroupa")
    if kind == "plummer":
        return c.pos, c.mass
    rng = np.random.default_rng(41)
    runs = [rng.normal(size=3) + np.zeros((k, 3)) for k in (9, 63, 64, 65, 129, 1025, 4097)]
    if kind == "point":
        runs, c.pos, c.mass = [np.zeros((1500, 3))], c.pos[:0], c.mass[:0]
    pos = np.concatenate(runs + [c.pos])
    return pos, rng.uniform(0.5, 1.5, pos.shape[0]) / pos.shape[0]


@pytest.mark.parametrize("kind,n_leaf,n_crit", [("point", 8, 64), ("runs", 8, 64), ("runs", 8, 32), ("runs", 8, 7),
                                                ("runs", 1, 1), ("plummer", 300, 64), ("plummer", 40, 8)])
def test_nodes_and_groups_of_long_leaves(kind, n_leaf, n_crit):
    from paper_2110_11658_amd.api import Pbh
    print(f"long leaves {kind} n_leaf={n_leaf} n_crit={n_crit}", flush=True)
    pos, mass = _points(kind)
    p = Pbh(0, leaf_size=n_leaf, n_crit=n_crit)
    p.build(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda())
    order, _, ni, nd = p.debug_tree()
    oorder, oi, od = oracle.tree_nodes(pos, mass, n_leaf=n_leaf, D=21)
    assert np.array_equal(order.astype(np.int64), oorder)
    assert np.array_equal(ni, oi) and np.array_equal(nd, od)
    gb, gc, gbox = p.debug_groups()
    ob, oc = oracle.groups(pos, mass, n_leaf=n_leaf, n_crit=n_crit)
    assert np.array_equal(gb.astype(np.int64), ob) and np.array_equal(gc.astype(np.int64), oc)
    xs = pos[oorder]
    lo = np.minimum.reduceat(xs, ob, axis=0)
    hi = np.maximum.reduceat(xs, ob, axis=0)
    assert np.array_equal(gbox, np.concatenate([lo, hi], axis=1))


# copies of each point and how far they lie apart: the same key; keys that differ in
# their last bits only, in short runs and in runs too long to insert
@pytest.mark.parametrize("n,copies,apart", [(5000, 100, 0.0), (5000, 9, 3e-7), (5000, 100, 3e-7), (40000, 30, 0.0),
                                            (40000, 100, 3e-7), (300000, 12, 3e-7), (300000, 100, 0.0)])
def test_order_of_points_many_times_over(n, copies, apart):
    from paper_2110_11658_amd.api import Pbh
    print(f"order n={n} copies={copies} apart={apart}", flush=True)
    rng = np.random.default_rng(n + copies)
    pos = np.repeat(ic.plummer(n // copies, seed=5).pos, copies, axis=0)
    pos = (pos + apart * rng.normal(size=pos.shape))[rng.permutation(pos.shape[0])]
    if copies == 9:   # equal keys among them as well
        pos[::2][:pos[1::2].shape[0]] = pos[1::2]
    p = Pbh(0)
    for again in range(2):   # the second time in key order
        mass = np.full(pos.shape[0], 1.0 / pos.shape[0])
        p.build(torch.from_numpy(np.ascontiguousarray(pos)).cuda(), torch.from_numpy(mass).cuda())
        order, keys, _, _ = p.debug_tree()
        assert np.array_equal(np.sort(order), np.arange(pos.shape[0]))
        by_caller = np.empty(pos.shape[0], dtype=np.uint64)
        by_caller[order] = keys
        assert np.array_equal(order, np.argsort(by_caller, kind="stable"))
        pos = pos[order]
