"""Neighbour lists through the staging rows (pbh_force): lists of several copy
tiles of 64 entries, blocks of 64 particles that are full, of one particle and
many, against the CPU oracle's brute-force lists (equal sets, exactly)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2110_11658_amd import ic

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0) if torch.cuda.is_available() else None


@pytest.mark.parametrize("n,nbar", [(64, 40.0), (65, 64.0), (705, 130.0), (2100, 300.0), (9000, 65.0)])
def test_lists_of_several_tiles(n, nbar):
    from paper_2110_11658_amd.api import Pbh
    print(f"lists n={n} nbar={nbar}", flush=True)
    c = ic.plummer(n, seed=51, masses="kroupa")
    r_out = ic.r_out_for_nbar(n, nbar)
    pos, mass = torch.from_numpy(c.pos).to(DEV), torch.from_numpy(c.mass).to(DEV)
    p = Pbh(0)
    p.build(pos, mass)
    _, _, off, idx = p.force(0.1 * r_out, r_out, 0.5, 1e-4)
    off, idx = off.cpu().numpy(), idx.cpu().numpy()
    o_off, o_idx = oracle.nbr_brute(c.pos, r_out)
    assert np.array_equal(off, o_off)
    for i in range(n):
        a, b = off[i], off[i + 1]
        assert np.array_equal(np.sort(idx[a:b]), np.sort(o_idx[a:b]))
