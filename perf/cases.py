"""The calls whose speed this repository is measured by, as a program that uses the library makes them.

Every case is a Plummer model (or an ensemble of them) in Henon units, drawn on the GPU from the seed:

step      tree build + regular force + neighbour lists of one cluster: what an N-body code does
          once per regular step (positions moved, so the tree is new every time)
field     tree build + regular force into the caller's buffers, no lists and no host wait
ensemble  the same as step for many independent clusters in one batched call
irregular F_I, its time derivative and Phi_I from the lists, for all particles or for a block of targets
core      core quantities (6 nearest neighbours of a sample) on the tree of the last build
hermite   block-step Hermite integration of F_I over one regular step
p3t       the whole loop: kick, Hermite, rebuild, force, kick
kdk       leapfrog under the regular force, steps replayed as one graph
"""
import ctypes as C
import math

import numpy as np
import torch

from paper_2110_11658_amd import ic
from paper_2110_11658_amd._lib import check
from paper_2110_11658_amd.api import Pbh

PLUMMER_A = 3.0 * math.pi / 16.0


def listed():
    return [
        # a small cluster, the size of a unit test or of a low-N production run: launches and latency
        {"name": "step_4k", "kind": "step", "n": 4096, "masses": "equal", "prec": "mixed", "theta": 0.5, "nbar": 64.0,
         "buffer": 0.0, "eps": 1e-4},
        # a very small system (an open cluster, or the remnant of one)
        {"name": "step_700", "kind": "step", "n": 700, "masses": "kroupa", "prec": "mixed", "theta": 0.5, "nbar": 32.0,
         "buffer": 0.0, "eps": 1e-4},
        # an ordinary globular-cluster run
        {"name": "step_128k", "kind": "step", "n": 131072, "masses": "kroupa", "prec": "mixed", "theta": 0.5, "nbar": 64.0,
         "buffer": 0.0, "eps": 1e-5},
        # the headline: a million stars
        {"name": "step_1m", "kind": "step", "n": 1048576, "masses": "kroupa", "prec": "mixed", "theta": 0.5, "nbar": 64.0,
         "buffer": 0.0, "eps": 1e-6},
        # a reference run in full precision with buffered lists, at a size that is no multiple of anything
        {"name": "step_fp64_100003", "kind": "step", "n": 100003, "masses": "two", "prec": "fp64", "theta": 0.4, "nbar": 24.0,
         "buffer": 0.25, "eps": 1e-5},
        # 64 clusters of 1e4 to 2e5 stars advanced together, the throughput run
        {"name": "ensemble_64", "kind": "ensemble", "clusters": 64, "nmin": 10000, "nmax": 200000, "masses": "kroupa",
         "prec": "mixed", "theta": 0.5, "nbar": 64.0, "eps": 1e-6},
        # neighbour force of every star, as after a regular step (start of an irregular integration, energies)
        {"name": "irregular_1m", "kind": "irregular", "n": 1048576, "masses": "kroupa", "nbar": 64.0, "eps": 1e-6,
         "targets": 0, "jerk": True, "pot": True},
        # neighbour force of one block of a block-step integrator on the host's side of the call
        {"name": "irregular_block", "kind": "irregular", "n": 131072, "masses": "kroupa", "nbar": 64.0, "eps": 1e-5,
         "targets": 777, "jerk": True, "pot": False},
        # core radius and density of a large model, every regular step
        {"name": "core_1m", "kind": "core", "n": 1048576, "masses": "kroupa"},
        # one regular step of the irregular integrator alone, with the paper's radii
        {"name": "hermite_16k", "kind": "hermite", "n": 16384, "masses": "equal", "eps": 1e-5},
        # the paper's own loop at its headline size, one regular step
        {"name": "p3t_1m", "kind": "p3t", "n": 1048576, "masses": "kroupa", "theta": 0.4, "eps": 1e-6},
        # leapfrog: eight steps in a graph
        {"name": "kdk_64k", "kind": "kdk", "n": 65536, "masses": "kroupa", "theta": 0.5, "nbar": 64.0, "eps": 1e-6,
         "steps": 8},
    ]


def _log_size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "field", "ensemble", "irregular", "irregular", "core", "hermite", "p3t", "kdk"])
    masses = rng.choice(["equal", "kroupa", "kroupa", "two"])
    eps = rng.choice([1e-4, 1e-5, 1e-6])
    if kind in ("step", "field"):
        prec = rng.choice(["mixed", "mixed", "fp64"])
        return {"kind": kind, "n": _log_size(rng, 500, 1e6 if prec == "mixed" else 4e5), "masses": masses, "prec": prec,
                "theta": rng.choice([0.4, 0.5, 0.6, 0.7]), "nbar": float(rng.choice([8, 24, 64])),
                "buffer": rng.choice([0.0, 0.0, 0.25]) if kind == "step" else 0.0, "eps": eps}
    if kind == "ensemble":
        lo = _log_size(rng, 300, 2e4)
        return {"kind": kind, "clusters": rng.randint(3, 70), "nmin": lo, "nmax": int(lo * rng.uniform(1.0, 5.0)),
                "masses": masses, "prec": "mixed", "theta": 0.5, "nbar": float(rng.choice([24, 64])), "eps": eps}
    if kind == "irregular":
        n = _log_size(rng, 2000, 1e6)
        return {"kind": kind, "n": n, "masses": masses, "nbar": float(rng.choice([8, 24, 64])), "eps": eps,
                "targets": rng.choice([0, _log_size(rng, 10, n / 2)]), "jerk": rng.random() < 0.7, "pot": rng.random() < 0.5}
    if kind == "core":
        return {"kind": kind, "n": _log_size(rng, 2000, 1e6), "masses": rng.choice(["kroupa", "two"])}
    if kind == "hermite":
        return {"kind": kind, "n": _log_size(rng, 1000, 2e5), "masses": masses, "eps": 1e-5}
    if kind == "p3t":
        return {"kind": kind, "n": _log_size(rng, 2000, 6e5), "masses": masses, "theta": rng.choice([0.4, 0.5]), "eps": 1e-5}
    return {"kind": kind, "n": _log_size(rng, 1000, 4e5), "masses": masses, "theta": 0.5, "nbar": 64.0, "eps": eps,
            "steps": rng.randint(1, 8)}


# ---------------------------------------------------------------- inputs
def _masses(n, kind, gen):
    dev = torch.device("cuda", 0)
    if kind == "equal":
        return torch.full((n,), 1.0 / n, dtype=torch.float64, device=dev)
    if kind == "two":   # every tenth star ten times as heavy
        m = torch.ones(n, dtype=torch.float64, device=dev)
        m[::10] = 10.0
        return m / m.sum()
    # Kroupa: dN/dm ~ m^-1.3 on [0.08, 0.5], m^-2.3 on [0.5, 100], continuous at 0.5
    w1 = (0.5 ** -0.3 - 0.08 ** -0.3) / -0.3
    w2 = 0.5 * (100.0 ** -1.3 - 0.5 ** -1.3) / -1.3
    u = torch.rand(n, dtype=torch.float64, device=dev, generator=gen)
    low = torch.rand(n, dtype=torch.float64, device=dev, generator=gen) < w1 / (w1 + w2)
    ml = (0.08 ** -0.3 + u * (0.5 ** -0.3 - 0.08 ** -0.3)) ** (-1.0 / 0.3)
    mh = (0.5 ** -1.3 + u * (100.0 ** -1.3 - 0.5 ** -1.3)) ** (-1.0 / 1.3)
    m = torch.where(low, ml, mh)
    return m / m.sum()


def _plummer(n, masses, gen):
    """(pos, vel, mass): Plummer sphere, G = M = 1, E = -1/4, centre of mass at rest at the origin."""
    dev = torch.device("cuda", 0)

    def rand():
        return torch.rand(n, dtype=torch.float64, device=dev, generator=gen)

    def direction():
        z = 1.0 - 2.0 * rand()
        phi = 2.0 * math.pi * rand()
        s = torch.sqrt(torch.clamp(1.0 - z * z, min=0.0))
        return torch.stack((s * torch.cos(phi), s * torch.sin(phi), z), dim=1)

    x = 1e-9 + rand() * (0.999 - 1e-9)          # enclosed mass, the far halo cut off
    r = 1.0 / torch.sqrt(x ** (-2.0 / 3.0) - 1.0)
    pos = direction() * (PLUMMER_A * r)[:, None]
    # v = q v_esc with q^2 ~ Beta(3/2, 9/2), the isotropic Plummer distribution
    g1 = torch._standard_gamma(torch.full((n,), 1.5, dtype=torch.float64, device=dev), generator=gen)
    g2 = torch._standard_gamma(torch.full((n,), 4.5, dtype=torch.float64, device=dev), generator=gen)
    speed = torch.sqrt(g1 / (g1 + g2)) * math.sqrt(2.0) * (1.0 + r * r) ** -0.25 / math.sqrt(PLUMMER_A)
    vel = direction() * speed[:, None]
    mass = _masses(n, masses, gen)
    pos -= (mass[:, None] * pos).sum(0)
    vel -= (mass[:, None] * vel).sum(0)
    return pos.contiguous(), vel.contiguous(), mass


def _sizes(case):
    c = case["clusters"]
    g = (case["nmax"] / case["nmin"])
    n = [int(round(case["nmin"] * g ** ((k + 0.5) / c))) for k in range(c)]
    return [n[(k * 37) % c] if math.gcd(37, c) == 1 else n[k] for k in range(c)]


def _radii(case):
    r_out = ic.r_out_for_nbar(case["n"], case["nbar"])
    return 0.1 * r_out, r_out


def _ptr(t):
    return C.c_void_p(t.data_ptr())


def _stream():
    return C.c_void_p(torch.cuda.current_stream().cuda_stream)


def _force_buffers(s, n, entries):
    """The caller's result arrays, kept from step to step; the lists' one with room to spare."""
    dev = s["pos"].device
    s["acc"] = torch.zeros((n, 3), dtype=torch.float64, device=dev)
    s["pot"] = torch.zeros(n, dtype=torch.float64, device=dev)
    if entries:
        s["off"] = torch.zeros(n + 1, dtype=torch.int64, device=dev)
        s["idx"] = torch.zeros(int(1.4 * entries) + 4096, dtype=torch.int32, device=dev)


def _gen(seed):
    return torch.Generator(device=torch.device("cuda", 0)).manual_seed(int(seed))


def prepare(case, seed):
    kind = case["kind"]
    gen = _gen(seed)
    s = dict(case)
    if kind == "ensemble":
        sizes = _sizes(case)
        parts = [_plummer(n, case["masses"], gen) for n in sizes]
        s["offsets"] = np.concatenate(([0], np.cumsum(sizes))).astype(np.int64)
        s["pos"] = torch.cat([p[0] for p in parts])
        s["mass"] = torch.cat([p[2] for p in parts])
        s["r_out"] = np.array([ic.r_out_for_nbar(n, case["nbar"]) for n in sizes])
        s["r_in"] = 0.1 * s["r_out"]
        _force_buffers(s, sum(sizes), sum(sizes) * case["nbar"])
        s["p"] = Pbh(0, prec=case["prec"])
        return s
    n = case["n"]
    s["pos"], s["vel"], s["mass"] = _plummer(n, case["masses"], gen)
    s["p"] = p = Pbh(0, prec=case.get("prec", "mixed"))
    if kind in ("step", "field", "irregular", "kdk"):
        s["r_in"], s["r_out"] = _radii(case)
    if kind in ("step", "field"):
        _force_buffers(s, n, n * case["nbar"] * (1.0 + case["buffer"]) ** 3 if kind == "step" else 0)
    elif kind == "irregular":
        p.build(s["pos"], s["mass"])
        _, _, s["off"], s["idx"] = p.force(s["r_in"], s["r_out"], 0.5, case["eps"])
        t = case["targets"]
        s["tgt"] = None if t == 0 else torch.randperm(n, device=s["pos"].device, generator=gen)[:t].to(torch.int32)
    elif kind == "core":
        k = ic.core_sample_size(n)
        s["sample"] = torch.sort(torch.randperm(n, device=s["pos"].device, generator=gen)[:k])[0].to(torch.int32)
        p.build(s["pos"], s["mass"])
    elif kind in ("hermite", "p3t"):
        r = ic.paper_radii(n)
        s["r_out"], s["r_in"] = r["r_cut"], 0.1 * r["r_cut"]
        s["r_buff"], s["dt_reg"] = r["r_buff"], r["dt_reg"]
        if kind == "hermite":
            p.build(s["pos"], s["mass"])
            s["fr"], _, s["off"], s["idx"] = p.force(s["r_in"], s["r_out"], 0.5, case["eps"], r_buff=s["r_buff"])
    if kind in ("hermite", "p3t", "kdk"):   # the integrators move the particles in place
        s["x"], s["v"] = torch.empty_like(s["pos"]), torch.empty_like(s["vel"])
    return s


def run(s):
    p, kind = s["p"], s["kind"]
    if kind == "step":
        p.build(s["pos"], s["mass"])
        check(p.ctx, p.L.pbh_force_buffered(
            p.ctx, _ptr(s["pos"]), _ptr(s["mass"]), s["r_in"], s["r_out"], s["buffer"] * s["r_out"], s["theta"], s["eps"],
            _ptr(s["acc"]), _ptr(s["pot"]), _ptr(s["off"]), _ptr(s["idx"]), s["idx"].numel(), None, _stream()))
        return s["acc"], s["pot"], s["off"], s["idx"]
    if kind == "field":
        p.build(s["pos"], s["mass"])
        p.force_into(s["r_in"], s["r_out"], s["theta"], s["eps"], s["acc"], s["pot"])
        return s["acc"], s["pot"]
    if kind == "ensemble":
        p.build_batched(s["offsets"], s["pos"], s["mass"])
        check(p.ctx, p.L.pbh_force_batched(
            p.ctx, _ptr(s["pos"]), _ptr(s["mass"]), C.c_void_p(s["r_in"].ctypes.data), C.c_void_p(s["r_out"].ctypes.data),
            s["theta"], s["eps"], _ptr(s["acc"]), _ptr(s["pot"]), _ptr(s["off"]), _ptr(s["idx"]), s["idx"].numel(), None,
            _stream()))
        return s["acc"], s["pot"], s["off"], s["idx"]
    if kind == "irregular":
        return p.irregular(s["pos"], s["vel"], s["mass"], s["r_in"], s["r_out"], s["eps"], s["off"], s["idx"],
                           targets=s["tgt"], jerk=s["jerk"], pot=s["pot"], validate=False)
    if kind == "core":
        return p.core(s["pos"], s["mass"], s["sample"])
    # every pass starts from the same model
    s["x"].copy_(s["pos"])
    s["v"].copy_(s["vel"])
    if kind == "hermite":
        info = p.hermite(s["x"], s["v"], s["mass"], s["fr"], s["r_in"], s["r_out"], s["eps"], s["off"], s["idx"], s["dt_reg"])
        return s["x"], s["v"], info
    if kind == "p3t":
        energy, info = p.p3t(s["x"], s["v"], s["mass"], s["r_in"], s["r_out"], s["r_buff"], s["theta"], s["eps"], s["dt_reg"])
        return s["x"], s["v"], energy, info
    energy = p.kdk(s["x"], s["v"], s["mass"], 1.0 / 1024.0, s["steps"], s["r_in"], s["r_out"], s["theta"], s["eps"])
    return s["x"], s["v"], energy


# ---------------------------------------------------------------- work
def _force_work(n, theta, nbar):
    """Interactions of one walk as the method needs them (a fit to counted walks of Plummer models:
    3300 multipoles a particle at 2^20 and theta = 0.5), 55 operations each, and 50 for each pair of a near leaf."""
    pn = min(3300.0 * (0.5 / theta) ** 2.1 * math.log2(max(n, 2)) / 20.0, float(n))
    return n * (55.0 * pn + 50.0 * min(10.0 * nbar, float(n)))


def work(case):
    kind = case["kind"]
    if kind == "ensemble":
        sizes = _sizes(case)
        n = sum(sizes)
        return {"bytes": n * (32 + 32 + 8 + 4 * case["nbar"]), "flops": sum(_force_work(k, case["theta"], case["nbar"]) for k in sizes)}
    n = case["n"]
    if kind == "step":
        nbar = case["nbar"] * (1.0 + case["buffer"]) ** 3
        return {"bytes": n * (32 + 32 + 8 + 4 * nbar), "flops": _force_work(n, case["theta"], nbar)}
    if kind == "field":
        return {"bytes": n * 64, "flops": _force_work(n, case["theta"], case["nbar"])}
    if kind == "irregular":
        t = case["targets"] or n
        pair = 40 + 33 * bool(case["jerk"]) + 22 * bool(case["pot"])
        out = 24 + 24 * bool(case["jerk"]) + 8 * bool(case["pot"])
        read = min(n, t * (1 + case["nbar"])) * (32 + 24 * bool(case["jerk"]))
        return {"bytes": read + t * (16 + 4 * case["nbar"] + out), "flops": t * case["nbar"] * pair}
    if kind == "core":
        k = ic.core_sample_size(n)
        return {"bytes": n * 32 + k * 12, "flops": n * 10 + k * 100 * 9}
    if kind == "hermite":   # about four steps a particle, two neighbours each
        return {"bytes": n * (24 * 5 + 8 + 8), "flops": n * 4.3 * 2 * 95}
    if kind == "p3t":
        return {"bytes": n * (24 * 4 + 8), "flops": 2 * _force_work(n, case["theta"], 1.6) + n * 4.3 * 2 * 95}
    return {"bytes": n * (24 * 4 + 8) * case["steps"], "flops": (case["steps"] + 1) * _force_work(n, case["theta"], case["nbar"])}


# ---------------------------------------------------------------- plain 64-bit values
def _changeover(r_in, r_out):
    """(W(s), Phi_R(s)) of the changeover split, dPhi_R/ds = W / s^2 and Phi_R = -1/s from r_out on."""
    d, a = r_out - r_in, r_in / (r_out - r_in)
    c = np.zeros(8)   # g(t - a) = sum c_k t^k with g(x) = 35 x^4 - 84 x^5 + 70 x^6 - 20 x^7
    for q, g in ((4, 35.0), (5, -84.0), (6, 70.0), (7, -20.0)):
        for k in range(q + 1):
            c[k] += g * math.comb(q, k) * (-a) ** (q - k)

    def prim(t, log):   # integral of g(t - a) / t^2
        v = -c[0] / t + c[1] * log(t)
        for k in range(2, 8):
            v = v + c[k] * t ** (k - 1) / (k - 1)
        return v

    top = prim(a + 1.0, math.log)
    inner = -1.0 / r_out - (top - prim(a, math.log)) / d

    def weight(s):
        x = ((s - r_in) / d).clamp(0.0, 1.0)
        return x ** 4 * (35.0 + x * (-84.0 + x * (70.0 - 20.0 * x)))

    def phi(s):
        t = s / d
        mid = -1.0 / r_out - (top - prim(t.clamp(min=a), torch.log)) / d
        return torch.where(s >= r_out, -1.0 / s, torch.where(s < r_in, torch.full_like(s, inner), mid))

    return weight, phi


def _direct(pos, mass, r_in, r_out, eps):
    weight, phi = _changeover(r_in, r_out)
    n = pos.shape[0]
    acc, pot = torch.empty_like(pos), torch.empty_like(mass)
    x, y, z = (pos[:, k].contiguous() for k in range(3))
    step = max(1, min(n, (1 << 26) // n))
    for a in range(0, n, step):
        b = min(n, a + step)
        dx, dy, dz = x[None, :] - x[a:b, None], y[None, :] - y[a:b, None], z[None, :] - z[a:b, None]
        s2 = dx * dx + dy * dy + dz * dz + eps * eps
        s = torch.sqrt(s2)
        f = mass[None, :] * weight(s) / (s2 * s)
        acc[a:b, 0], acc[a:b, 1], acc[a:b, 2] = (f * dx).sum(1), (f * dy).sum(1), (f * dz).sum(1)
        ph = mass[None, :] * phi(s)
        ph[torch.arange(b - a, device=pos.device), torch.arange(a, b, device=pos.device)] = 0.0
        pot[a:b] = ph.sum(1)
    return acc, pot


def _exact_irregular(s):
    weight, phi = _changeover(s["r_in"], s["r_out"])
    off, idx = s["off"], s["idx"].long()
    tgt = torch.arange(s["n"], device=idx.device) if s["tgt"] is None else s["tgt"].long()
    acc, jerk = (torch.zeros((tgt.numel(), 3), dtype=torch.float64, device=idx.device) for _ in range(2))
    pot = torch.zeros(tgt.numel(), dtype=torch.float64, device=idx.device)
    d = s["r_out"] - s["r_in"]
    for a in range(0, tgt.numel(), 1 << 17):
        t = tgt[a:a + (1 << 17)]
        cnt = off[t + 1] - off[t]
        row = torch.repeat_interleave(torch.arange(t.numel(), device=idx.device), cnt)
        first = torch.cumsum(cnt, 0) - cnt
        j = idx[off[t][row] + torch.arange(row.numel(), device=idx.device) - first[row]]
        i = t[row]
        dr, m = s["pos"][j] - s["pos"][i], s["mass"][j]
        s2 = (dr * dr).sum(1) + s["eps"] ** 2
        q = torch.sqrt(s2)
        k = torch.where(q < s["r_out"], 1.0 - weight(q), torch.zeros_like(q))
        acc[a:a + t.numel()].index_add_(0, row, (m * k / (s2 * q))[:, None] * dr)
        if s["jerk"]:
            u = s["vel"][j] - s["vel"][i]
            du = (dr * u).sum(1)
            x = ((q - s["r_in"]) / d).clamp(0.0, 1.0)
            kd = -140.0 * x ** 3 * (1.0 - x) ** 3 * du / (q * d)
            term = (m * k / (s2 * q))[:, None] * (u - (3.0 * du / s2)[:, None] * dr) + (m * kd / (s2 * q))[:, None] * dr
            jerk[a:a + t.numel()].index_add_(0, row, term)
        if s["pot"]:
            pot[a:a + t.numel()].index_add_(0, row, m * (-1.0 / q - phi(q)))
    return acc, jerk if s["jerk"] else None, pot if s["pot"] else None


def _exact_core(s):
    pos, mass, sample = s["pos"], s["mass"], s["sample"].long()
    n = pos.shape[0]
    rho = torch.empty(sample.numel(), dtype=torch.float64, device=pos.device)
    step = max(1, (1 << 26) // n)
    for a in range(0, sample.numel(), step):
        i = sample[a:a + step]
        r2 = torch.zeros((i.numel(), n), dtype=torch.float64, device=pos.device)
        for k in range(3):
            r2 += (pos[i, k][:, None] - pos[:, k][None, :]) ** 2
        r2[torch.arange(i.numel(), device=pos.device), i] = math.inf
        v, j = torch.topk(r2, 6, dim=1, largest=False, sorted=True)
        rho[a:a + step] = mass[j[:, :5]].sum(1) / (4.0 * math.pi / 3.0 * v[:, 5] ** 1.5)
    x = pos[sample]
    center = (rho[:, None] * x).sum(0) / rho.sum()
    w = rho * rho
    rho_core = float(w.sum() / rho.sum())
    r_core = float(torch.sqrt((w * ((x - center) ** 2).sum(1)).sum() / w.sum()))
    r, order = torch.sort(torch.sqrt(((pos - center) ** 2).sum(1)))
    cum = torch.cumsum(mass[order], 0)
    r_half = float(r[int(torch.searchsorted(cum, 0.5 * cum[-1]))])
    r_min = 4.0 * r_half / (n * rho_core ** (1.0 / 3.0))
    return rho, {"center": center.cpu().numpy(), "rho_core": rho_core, "r_core": r_core, "n_core": None, "r_half": r_half,
                 "r_min": r_min, "dt_min": 0.01 * math.sqrt(r_min ** 3)}


def exact(case, seed):
    """Direct sums, brute-force neighbours and plain leapfrog where the pairs can be counted out; the block-step
    integration (hermite, p3t) is defined by its own scheme and has no other value."""
    kind = case["kind"]
    if kind in ("step", "field"):
        if case["n"] > 140000:
            return None
        s = prepare(case, seed)
        acc, pot = _direct(s["pos"], s["mass"], s["r_in"], s["r_out"], s["eps"])
        return (acc, pot) if kind == "field" else (acc, pot, None, None)
    if kind == "ensemble":
        if sum(n * n for n in _sizes(case)) > 2e10:
            return None
        s = prepare(case, seed)
        acc, pot = torch.empty_like(s["pos"]), torch.empty_like(s["mass"])
        for k in range(case["clusters"]):
            a, b = int(s["offsets"][k]), int(s["offsets"][k + 1])
            acc[a:b], pot[a:b] = _direct(s["pos"][a:b], s["mass"][a:b], s["r_in"][k], s["r_out"][k], s["eps"])
        return acc, pot, None, None
    if kind == "irregular":
        return _exact_irregular(prepare(case, seed))
    if kind == "core":
        return _exact_core(prepare(case, seed)) if case["n"] <= 400000 else None
    if kind == "kdk":
        n, h = case["n"], 1.0 / 1024.0
        if n * n * (case["steps"] + 1.0) > 6e10:
            return None
        s = prepare(case, seed)
        x, v, m = s["pos"].clone(), s["vel"].clone(), s["mass"]
        acc, pot = _direct(x, m, s["r_in"], s["r_out"], s["eps"])
        energy = [0.5 * (m * (v * v).sum(1)).sum() + 0.5 * (m * pot).sum()]
        for _ in range(case["steps"]):
            v += 0.5 * h * acc
            x += h * v
            acc, pot = _direct(x, m, s["r_in"], s["r_out"], s["eps"])
            v += 0.5 * h * acc
            energy.append(0.5 * (m * (v * v).sum(1)).sum() + 0.5 * (m * pot).sum())
        return x, v, torch.stack(energy)
    return None
