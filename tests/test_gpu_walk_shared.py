"""Groups of a walk that two waves share: which ones are shared depends on how
many groups the whole walk has, and the results must not. One cluster is walked
alone (every group shared) and as the first, the middle and the last of an
ensemble that makes the walk share some of its groups, or none; force, potential
and lists are the same bit for bit, with and without neighbour lists.
"""
import numpy as np
import pytest
import torch

from paper_2110_11658_amd import ic

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# n_crit 8: about one group to 4 particles; 512 waves a queue share all groups
# up to 320 a queue, some up to 4096, none beyond
@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("filler", [2, 4, 40, 330])
def test_results_do_not_depend_on_the_sharing(prec, filler):
    from paper_2110_11658_amd.api import Pbh
    kw = dict(prec=prec, key_bits=18, n_crit=8)
    a = ic.plummer(2900, seed=3, masses="kroupa")
    r_in, r_out, theta, eps = 0.006, 0.06, 0.5, 1e-5
    alone = Pbh(0, **kw)
    alone.build(_t(a.pos), _t(a.mass))
    acc, pot, off, idx = (t.cpu().numpy() for t in alone.force(r_in, r_out, theta, eps))
    b = ic.plummer(3100, seed=4, masses="kroupa")
    clusters = [a] + [b] * (filler // 2) + [a] + [b] * (filler - filler // 2) + [a]
    offsets = np.concatenate(([0], np.cumsum([c.n for c in clusters])))
    pos, mass = np.concatenate([c.pos for c in clusters]), np.concatenate([c.mass for c in clusters])
    p = Pbh(0, **kw)
    p.build_batched(offsets, _t(pos), _t(mass))
    n = len(clusters)
    ri, ro = [r_in] * n, [r_out] * n
    print(f"shared {prec} filler={filler}", flush=True)
    for lists in (True, False):
        ga, gp, go, gi = p.force_batched(ri, ro, theta, eps, neighbours=lists)
        print("groups", p.stats()["n_groups"], flush=True)
        ga, gp = ga.cpu().numpy(), gp.cpu().numpy()
        go, gi = (go.cpu().numpy(), gi.cpu().numpy()) if lists else (None, None)
        for k in [i for i, c in enumerate(clusters) if c is a]:
            s = slice(offsets[k], offsets[k + 1])
            assert np.array_equal(ga[s], acc) and np.array_equal(gp[s], pot)
            if lists:
                assert np.array_equal(go[s.start:s.stop + 1] - go[s.start], off)
                assert np.array_equal(gi[go[s.start]:go[s.stop]], idx + s.start)


@pytest.mark.parametrize("n,n_crit,theta,r_out", [(2, 64, 0.5, 0.1), (64, 64, 0.5, 2.0), (700, 64, 0.0, 0.1),
                                                  (2900, 64, 0.5, 0.06), (2900, 48, 0.7, 0.3), (900, 64, 0.5, 9.0)])
def test_four_waves_a_group_equal_one(n, n_crit, theta, r_out):
    # a walk of few particles gives four waves to a group, of many one: the
    # cluster alone and in an ensemble of more than 40960 particles, bit for bit
    # (far, near and multipole tiles missing or many, lists that overflow their rows)
    from paper_2110_11658_amd.api import Pbh
    kw = dict(prec="mixed", key_bits=18, n_crit=n_crit)
    a, b = ic.plummer(n, seed=5, masses="kroupa"), ic.plummer(45000, seed=6)
    r_in, eps = 0.1 * r_out, 1e-5
    print(f"team n={n} n_crit={n_crit} theta={theta} r_out={r_out}", flush=True)
    alone, p = Pbh(0, **kw), Pbh(0, **kw)
    alone.build(_t(a.pos), _t(a.mass))
    acc, pot, off, idx = (t.cpu().numpy() for t in alone.force(r_in, r_out, theta, eps))
    offsets = np.array([0, n, n + b.n])
    p.build_batched(offsets, _t(np.concatenate([a.pos, b.pos])), _t(np.concatenate([a.mass, b.mass])))
    ga, gp, go, gi = (t.cpu().numpy() for t in p.force_batched([r_in, 0.001], [r_out, 0.01], theta, eps))
    assert np.array_equal(ga[:n], acc) and np.array_equal(gp[:n], pot)
    assert np.array_equal(go[:n + 1], off) and np.array_equal(gi[:off[-1]], idx)
    ga, gp, _, _ = alone.force(r_in, r_out, theta, eps, neighbours=False)
    assert np.array_equal(ga.cpu().numpy(), acc) and np.array_equal(gp.cpu().numpy(), pot)
