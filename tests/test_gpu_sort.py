"""The key sort of a build (and of the half-mass radius): the exported order of
a build is the stable order of its exported keys, whatever the keys look like.

Sizes around the sort's dispatch: one workgroup up to 8192 keys; tiles of 512,
2048 and 4096 keys from there, the last tile full, short by one and with one
key. Inputs: a Plummer model; a model in caller order already sorted by key; all
points coincident; half of them in one point; a tight cluster with one far
particle, whose keys agree in nearly all of the digits that are sorted first.
"""
import numpy as np
import pytest
import torch

from paper_2110_11658_amd import ic

pytestmark = pytest.mark.gpu


def _positions(kind, n):
    rng = np.random.default_rng(n)
    pos = rng.normal(size=(n, 3))
    if kind == "plummer":
        pos = ic.plummer(n, seed=7).pos
    elif kind == "coincident":
        pos[:] = pos[0]
    elif kind == "half":
        pos[rng.permutation(n)[: n // 2]] = pos[0]
    elif kind == "escaper":
        pos *= 1e-6
        pos[n // 3] = (3e5, -2e5, 1e5)
    return pos


@pytest.mark.parametrize("n,kinds", [
    (1, ("plummer",)), (2, ("plummer", "coincident")), (1023, ("plummer", "half")),
    (8192, ("plummer", "coincident", "half", "escaper")), (8193, ("plummer", "coincident", "half", "escaper")),
    (20000, ("plummer", "half", "escaper")), (262144, ("plummer", "coincident")), (262145, ("plummer", "escaper")),
    (524289, ("plummer", "half")), (1048577, ("plummer",)), (4194304, ("plummer",)), (4194305, ("plummer",)),
])
def test_order_is_the_stable_order_of_the_keys(n, kinds):
    from paper_2110_11658_amd.api import Pbh
    for kind in kinds:
        print(f"sort {kind} n={n}", flush=True)
        pos = _positions(kind, n)
        mass = np.full(n, 1.0 / n)
        p = Pbh(0)
        for again in range(2):   # the second time in key order
            x, m = torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda()
            p.build(x, m)
            order, keys, _, _ = p.debug_tree()
            assert np.array_equal(np.sort(order), np.arange(n))
            by_caller = np.empty(n, dtype=np.uint64)
            by_caller[order] = keys
            assert np.array_equal(order, np.argsort(by_caller, kind="stable"))
            pos = np.ascontiguousarray(pos[order])
        p.close()
