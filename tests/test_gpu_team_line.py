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
