"""Walks with tiles of 96 and 128 entries: which groups two waves share depends on the
number of groups a wave, and the results must not. One cluster alone (every group
shared) and in ensembles that share some of its groups, or none, bit for bit.
"""
import numpy as np
import pytest
import torch

from paper_2110_11658_amd import ic

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# n_crit 8: about one group to 4 particles; 320 and 384 waves a queue share some groups
# up to 1.5 a wave (tiles of 128) and 8 a wave (96)
@pytest.mark.parametrize("tile", [96, 128])
@pytest.mark.parametrize("filler", [2, 4, 6, 40])
def test_results_do_not_depend_on_the_sharing(tile, filler):
    from paper_2110_11658_amd.api import Pbh
    kw = dict(prec="mixed", key_bits=18, n_crit=8, walk_tile=tile)
    a, b = ic.plummer(2900, seed=3, masses="kroupa"), ic.plummer(3100, seed=4, masses="kroupa")
    r_in, r_out, theta, eps = 0.006, 0.06, 0.5, 1e-5
    alone, p = Pbh(0, **kw), Pbh(0, **kw)
    alone.build(_t(a.pos), _t(a.mass))
    acc, pot, off, idx = (t.cpu().numpy() for t in alone.force(r_in, r_out, theta, eps))
    clusters = [a] + [b] * filler + [a]
    offsets = np.concatenate(([0], np.cumsum([c.n for c in clusters])))
    p.build_batched(offsets, _t(np.concatenate([c.pos for c in clusters])),
                    _t(np.concatenate([c.mass for c in clusters])))
    n = len(clusters)
    ga, gp, go, gi = (t.cpu().numpy() for t in p.force_batched([r_in] * n, [r_out] * n, theta, eps))
    print(f"tile {tile} filler {filler} groups {p.stats()['n_groups']}", flush=True)
    for k in (0, n - 1):
        s = slice(offsets[k], offsets[k + 1])
        assert np.array_equal(ga[s], acc) and np.array_equal(gp[s], pot)
        assert np.array_equal(go[s.start:s.stop + 1] - go[s.start], off)
        assert np.array_equal(gi[go[s.start]:go[s.stop]], idx + s.start)
    alone.close()
    p.close()
