"""Nodes and moments of builds around the sizes where the nodes that straddle
tiles of particles take another launch or wider workgroups (1024, 65536, 131072
particles): structure, boxes, centres and quadrupoles equal the CPU oracle's bit
for bit (same FP64 operation order)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2110_11658_amd import ic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_leaf", [(1024, 8), (1025, 8), (65536, 8), (65537, 16), (100003, 8), (131072, 8),
                                      (131073, 16)])
def test_tree_at_the_straddling_launches(n, n_leaf):
    from paper_2110_11658_amd.api import Pbh
    print(f"tree n={n} n_leaf={n_leaf}", flush=True)
    c = ic.plummer(n, seed=31, masses="kroupa")
    p = Pbh(0, leaf_size=n_leaf)
    p.build(torch.from_numpy(c.pos).cuda(), torch.from_numpy(c.mass).cuda())
    order, keys, ni, nd = p.debug_tree()
    oorder, oi, od = oracle.tree_nodes(c.pos, c.mass, n_leaf=n_leaf, D=21)
    assert np.array_equal(order.astype(np.int64), oorder)
    assert np.array_equal(ni, oi) and np.array_equal(nd, od)
