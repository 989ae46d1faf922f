"""Rounds of the irregular force in key order: 2, 3 or 6 list entries a lane, by the
list buffer's entries a particle and by what is left of the lists of a wave. The
lanes sum their entries in list order on every route, so the sums equal those of
the caller-array route (a context without a build) bit for bit."""
import numpy as np
import pytest
import torch

from paper_2110_11658_amd import ic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths", ["none", "one", "ragged", "rounds"])
@pytest.mark.parametrize("jerk,pot", [(False, False), (False, True), (True, False), (True, True)])
def test_rounds_do_not_change_the_sums(lengths, jerk, pot):
    from paper_2110_11658_amd.api import Pbh
    print(f"irregular rounds {lengths} jerk={jerk} pot={pot}", flush=True)
    n = 3001
    c = ic.plummer(n, seed=9, masses="kroupa")
    rng = np.random.default_rng(9)
    k = np.arange(n)
    # one long list among short ones, and lengths at the ends of rounds of 2, 3 and 6
    cnt = {"none": 0 * k, "one": np.where(k == 1700, 1000, 0), "ragged": (7 * k) % 61,
           "rounds": np.array([0, 1, 8, 9, 15, 16, 17, 24, 25, 47, 48, 49, 64, 65])[k % 14]}[lengths]
    off = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int64)
    idx = rng.integers(0, n, max(int(off[-1]), 1)).astype(np.int32)   # (a particle's own index too)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    pos, vel, mass, toff = t(c.pos), t(c.vel), t(c.mass), t(off)
    built, plain = Pbh(0), Pbh(0)
    built.build(pos, mass)
    for entries in (16 * n, 16 * n + 1, 40 * n, 40 * n + 1):   # the buffer, whatever the lists hold
        if entries < idx.size:
            continue
        buf = t(np.concatenate([idx, np.zeros(entries - idx.size, dtype=np.int32)]))
        got = built.irregular(pos, vel, mass, 0.02, 0.2, 1e-4, toff, buf, jerk=jerk, pot=pot)
        ref = plain.irregular(pos, vel, mass, 0.02, 0.2, 1e-4, toff, buf, jerk=jerk, pot=pot)
        for a, b in zip(got, ref):
            assert (a is None and b is None) or torch.equal(a, b)
