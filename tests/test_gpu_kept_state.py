"""What a context keeps between calls follows the parameters of the call at hand."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2110_11658_amd import ic

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _p(t):
    return C.c_void_p(t.data_ptr())


@pytest.mark.parametrize("change", [dict(walk_tile=128), dict(lanes_per_particle=1)])
def test_leapfrog_graph_takes_new_walk_parameters(change):
    # the same arrays before and after the change: a graph captured with the former
    # tile or lanes must not be replayed
    from paper_2110_11658_amd.api import Pbh
    print(f"leapfrog, then {change}, then again", flush=True)
    c = ic.plummer(3000, seed=41, masses="kroupa")
    pos, vel, mass = _t(c.pos), _t(c.vel), _t(c.mass)
    energy = torch.empty(4, dtype=torch.float64, device="cuda")

    def leapfrog(p):
        pos.copy_(_t(c.pos))
        vel.copy_(_t(c.vel))
        st = p.L.pbh_kdk_graph(p.ctx, c.n, _p(pos), _p(vel), _p(mass), 1.0 / 256, 3, 0.01, 0.1, 0.5, 1e-3, _p(energy),
                               C.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == 0
        torch.cuda.synchronize()
        return [t.cpu().numpy().copy() for t in (pos, vel, energy)]

    kept, fresh = Pbh(0), Pbh(0, **change)
    first = leapfrog(kept)
    kept.set_params(**change)
    second, want = leapfrog(kept), leapfrog(fresh)
    assert not np.array_equal(first[1], want[1])   # (the parameter is seen in the sums' rounding)
    for a, b in zip(second, want):
        assert np.array_equal(a, b)
    kept.close()
    fresh.close()


def test_refused_leapfrog_leaves_no_build():
    # more particles than node indices can name: refused once the sizes are set. The
    # tree of the build before must not be walked with them
    from paper_2110_11658_amd import _lib
    from paper_2110_11658_amd.api import Pbh
    print("leapfrog refused, then a force of the build before", flush=True)
    c = ic.plummer(1000, seed=42, masses="kroupa")
    pos, vel, mass = _t(c.pos), _t(c.vel), _t(c.mass)
    p = Pbh(0)
    p.build(pos, mass)
    want = [t.cpu().numpy() for t in p.force(0.01, 0.1, 0.5, 1e-3)]
    energy = torch.empty(2, dtype=torch.float64, device="cuda")
    st = p.L.pbh_kdk_graph(p.ctx, (1 << 31) - 2, _p(pos), _p(vel), _p(mass), 1.0 / 256, 1, 0.01, 0.1, 0.5, 1e-3,
                           _p(energy), C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == _lib.PBH_E_ARG
    with pytest.raises(_lib.PbhError) as e:
        p.force(0.01, 0.1, 0.5, 1e-3)
    assert e.value.status == _lib.PBH_E_STATE
    p.build(pos, mass)
    for a, b in zip(p.force(0.01, 0.1, 0.5, 1e-3), want):
        assert np.array_equal(a.cpu().numpy(), b)
    p.close()


def test_hermite_after_its_buffers_were_replaced():
    # a call that ends between the allocation of larger Hermite buffers and the capture
    # of its batch: the batch captured before must not be replayed on the freed ones
    from paper_2110_11658_amd import _lib
    from paper_2110_11658_amd.api import Pbh
    print("hermite, a refused p3t of more particles, hermite", flush=True)
    c, big = ic.plummer(700, seed=43, masses="kroupa"), ic.plummer(2000, seed=44, masses="kroupa")
    r_out = ic.r_out_for_nbar(c.n, 12.0)
    r_in, eps = 0.1 * r_out, 1e-4
    pos, vel, mass = _t(c.pos), _t(c.vel), _t(c.mass)
    p = Pbh(0, prec="fp64")
    p.build(pos, mass)
    fr, _, off, idx = p.force(r_in, r_out, 0.0, eps, r_buff=0.5 * r_out)

    def hermite():
        pos.copy_(_t(c.pos))
        vel.copy_(_t(c.vel))
        st = p.hermite(pos, vel, mass, fr, r_in, r_out, eps, off, idx, 1.0 / 256)
        torch.cuda.synchronize()
        return pos.cpu().numpy(), vel.cpu().numpy(), st

    first = hermite()
    bad = big.pos.copy()
    bad[1234, 1] = np.nan
    with pytest.raises(_lib.PbhError) as e:
        p.p3t(_t(bad), _t(big.vel), _t(big.mass), r_in, r_out, 0.5 * r_out, 0.5, eps, 1.0 / 256, 1)
    assert e.value.status == _lib.PBH_E_NONFINITE
    again = hermite()
    assert np.array_equal(first[0], again[0]) and np.array_equal(first[1], again[1]) and first[2] == again[2]
    p.close()
