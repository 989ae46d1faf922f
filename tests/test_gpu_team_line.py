"""Teams of four waves a group and ensembles of small clusters, on both sides of the
line between a team and one wave a group (48 times as many particles in each as there
are clusters): the route by the walk's grid, and results equal to those of each cluster
built alone, bit for bit.
"""
import numpy as np
import pytest
import torch

from paper_2110_11658_amd import ic

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _grid(p):
    return len(p.debug_wave_log()[0])


@pytest.mark.parametrize("sizes,team", [
    ([47], False), ([48], True), ([95, 95], False), ([96, 96], True), ([239] * 5, False), ([240] * 5, True),
    ([20] * 300, False), ([1] * 50, False), ([7] * 40 + [3000], True), ([7, 1, 2], False)])
def test_team_line_of_ensembles(sizes, team):
    from paper_2110_11658_amd.api import Pbh
    print(f"{len(sizes)} clusters of {min(sizes)} to {max(sizes)}, team {team}", flush=True)
    kw = dict(prec="mixed", key_bits=18, n_crit=32)
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    c = ic.plummer(int(offsets[-1]), seed=21, masses="kroupa")
    pos, mass, k = c.pos, c.mass, len(sizes)
    r_in, r_out, theta, eps = 0.05, 0.5, 0.5, 1e-5
    ref, p = Pbh(0, **kw), Pbh(0, **kw)
    one = ic.plummer(2000, seed=22)
    ref.build(_t(one.pos), _t(one.mass))
    ref.force(r_in, r_out, theta, eps)
    p.build_batched(offsets, _t(pos), _t(mass))
    acc, pot, off, idx = (t.cpu().numpy() for t in p.force_batched([r_in] * k, [r_out] * k, theta, eps))
    assert (_grid(p) == _grid(ref)) == team
    for q in sorted({0, 1, k // 2, k - 1} & set(range(k))):
        s = slice(offsets[q], offsets[q + 1])
        ref.build(_t(pos[s]), _t(mass[s]))
        a, f, o, i = (t.cpu().numpy() for t in ref.force(r_in, r_out, theta, eps))
        assert np.array_equal(acc[s], a) and np.array_equal(pot[s], f)
        assert np.array_equal(off[s.start:s.stop + 1] - off[s.start], o)
        assert np.array_equal(idx[off[s.start]:off[s.stop]], i + s.start)
    ref.close()
    p.close()


@pytest.mark.parametrize("n,leaf,team", [(2600, 2048, True), (2600, 2049, False), (2048, 100000, True),
                                         (2049, 100000, False)])
def test_team_line_of_large_leaves(n, leaf, team):
    # (an ensemble of more than 40960 particles takes one wave a group)
    from paper_2110_11658_amd.api import Pbh
    print(f"{n} particles in leaves of up to {leaf}, team {team}", flush=True)
    kw = dict(prec="mixed", key_bits=18, n_crit=32, leaf_size=leaf)
    c, big, one = ic.plummer(n, seed=23, masses="kroupa"), ic.plummer(41000, seed=24), ic.plummer(2000, seed=22)
    r_in, r_out, theta, eps = 0.01, 0.1, 0.5, 1e-5
    ref, p, q = Pbh(0, prec="mixed"), Pbh(0, **kw), Pbh(0, **kw)
    ref.build(_t(one.pos), _t(one.mass))
    ref.force(r_in, r_out, theta, eps)
    p.build(_t(c.pos), _t(c.mass))
    acc, pot, off, idx = (t.cpu().numpy() for t in p.force(r_in, r_out, theta, eps))
    assert (_grid(p) == _grid(ref)) == team
    q.build_batched([0, n, n + big.n], _t(np.concatenate([c.pos, big.pos])), _t(np.concatenate([c.mass, big.mass])))
    a, f, o, i = (t.cpu().numpy() for t in q.force_batched([r_in, 0.0], [r_out, 0.001], theta, eps))
    assert np.array_equal(a[:n], acc) and np.array_equal(f[:n], pot)
    assert np.array_equal(o[:n + 1], off) and np.array_equal(i[:o[n]], idx)
    for h in (ref, p, q):
        h.close()
