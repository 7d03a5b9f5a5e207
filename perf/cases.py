"""Workloads of the Kob-Andersen MD library as its users run them, for timing.

Every case is one pass through the public entry points (``md.System``) on a
liquid configuration made from a seed alone: a small periodic box is melted
and thermalised by a plain torch MD loop, tiled to the size of the case,
thinned at random to the exact particle numbers and given fresh
Maxwell-Boltzmann velocities.

Kinds of pass (``op``):
  nve     ``steps`` velocity-Verlet steps, by the eager call or as a replay of
          a captured graph; the outputs are the whole exported state
  bath    the same with the stochastic Maxwell-Boltzmann bath
  nose    the same with the Nose-Hoover bath
  forces  cells, neighbour lists, forces, potential energy and virial of a
          given configuration
  rdf     the pair-distance histogram
  move    mean-square displacement and self van Hove histogram against a
          stored origin
"""
import math

import numpy as np
import torch

from paper_2001_07089_amd import md
from paper_2001_07089_amd import workload as W

STATE = ("x", "y", "z", "vx", "vy", "vz", "ax", "ay", "az")
FLOP_PER_PAIR = 19
N_LARGE = 1 << 20


def _case(name, op, n, precision="fp64", rho=1.2, T=1.0, n_rep=1, n_max=0, T_max=0.0, skin=0.3, steps=0, graph=False,
          every=0, rmax=0.0, bins=0):
    """n: particles of a replica (with n_max > 0: sizes spread over [n, n_max]); T_max likewise."""
    c = dict(op=op, n=n, precision=precision, rho=rho, T=T, n_rep=n_rep, n_max=n_max, T_max=T_max, skin=skin,
             steps=steps, graph=graph, every=every, rmax=rmax, bins=bins)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the paper's own system (N = 1000, FP64), driven one step per call by
        # a program that looks at the state after every step
        _case("nve_1000_fp64_one_step", "nve", 1000, "fp64", T=2.0, steps=1),
        # the same system as most runs take it: many steps per call
        _case("nve_1000_fp64", "nve", 1000, "fp64", T=2.0, steps=50),
        # a temperature ladder's equilibration: 64 independent N = 1000
        # systems under the stochastic bath
        _case("bath_64x1000_fixed", "bath", 1000, "mixed_fixed", T=0.5, T_max=3.0, n_rep=64, steps=50, every=10),
        # the medium system's production run, replayed from a graph
        _case("nve_32000_mixed", "nve", 32000, "mixed", T=0.5, steps=50, graph=True),
        # the medium system under the Nose-Hoover bath, in FP64
        _case("nose_32000_fp64", "nose", 32000, "fp64", T=0.5, steps=20),
        # the headline benchmark: N = 2^20, 64-bit fixed-point force sums
        _case("nve_1048576_fixed", "nve", N_LARGE, "mixed_fixed", T=0.45, steps=20, graph=True),
        # the same system in FP64
        _case("nve_1048576_fp64", "nve", N_LARGE, "fp64", T=0.45, steps=20, graph=True),
        # the replica batch: 256 systems of 250 to 8000 particles
        _case("nve_batch256_mixed", "nve", 250, "mixed", T=0.45, T_max=2.0, n_rep=256, n_max=8000, steps=20,
              graph=True),
        # a configuration handed in from outside, of an odd size: lists,
        # forces, energy and virial
        _case("forces_100003_fixed", "forces", 100003, "mixed_fixed", T=0.8),
        # the medium system's histogram to half the box
        _case("rdf_32000_half_box", "rdf", 32000, "mixed", T=0.5, rmax=14.9, bins=200),
        # the large system's histogram over the first shells
        _case("rdf_1048576", "rdf", N_LARGE, "mixed_fixed", T=0.45, rmax=5.0, bins=200),
        # displacement measurements of a large odd-sized run
        _case("move_262147_mixed", "move", 262147, "mixed", T=0.5, bins=200),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["nve", "nve", "nve", "batch", "bath", "nose", "forces", "rdf", "move"])
    prec = rng.choice(["fp64", "mixed", "mixed_fixed"])
    rho = rng.choice([1.1, 1.2, 1.3])
    T = rng.uniform(0.45, 2.0)
    skin = rng.choice([0.2, 0.3, 0.3, 0.4])
    if op == "nve":
        n = _log_int(rng, 500, N_LARGE)
        steps = rng.randint(1, max(2, min(50, 20 * N_LARGE // n)))
        return _case("", "nve", n, prec, rho, T, skin=skin, steps=steps, graph=rng.random() < 0.5)
    if op == "batch":
        n_rep = _log_int(rng, 2, 256)
        return _case("", "nve", 250, prec, 1.2, 0.45, n_rep=n_rep, n_max=rng.randint(500, 8000), T_max=2.0, skin=skin,
                     steps=rng.randint(2, 20), graph=rng.random() < 0.5)
    if op == "bath":
        every = rng.randint(2, 20)
        return _case("", "bath", _log_int(rng, 400, 10000), prec, rho, 0.5, n_rep=rng.randint(1, 32), T_max=3.0, skin=skin,
                     steps=every * rng.randint(1, 3), every=every, graph=rng.random() < 0.5)
    if op == "nose":
        return _case("", "nose", _log_int(rng, 500, 200000), prec, rho, T, skin=skin, steps=rng.randint(1, 20),
                     graph=rng.random() < 0.5)
    if op == "forces":
        return _case("", "forces", _log_int(rng, 500, N_LARGE), prec, rho, T, skin=skin)
    if op == "rdf":
        n = _log_int(rng, 500, 400000)
        half = 0.49 * W.box_for(n, rho)
        # ordinary ranges, and half the box where that is still affordable
        rmax = half if n <= 32000 and rng.random() < 0.5 else min(half, rng.uniform(2.5, 6.0))
        return _case("", "rdf", n, prec, rho, T, rmax=rmax, bins=rng.randint(25, 500))
    return _case("", "move", _log_int(rng, 500, N_LARGE), prec, rho, T, bins=rng.randint(50, 500))


# ------------------------------------------------------------------ inputs
def _replicas(case):
    """(n, n_a, box, T) of every replica."""
    nr = case["n_rep"]
    if case["n_max"] > 0:
        rng = np.random.default_rng(W.BASE_SEED + 4000)
        ns = rng.integers(case["n"], case["n_max"] + 1, size=nr)
    else:
        ns = np.full(nr, case["n"])
    Ts = np.linspace(case["T"], case["T_max"], nr) if case["T_max"] > 0 else np.full(nr, case["T"])
    return [(int(n), W.n_a_for(int(n)), W.box_for(int(n), case["rho"]), float(T)) for n, T in zip(ns, Ts)]


def _pair_tables(is_b, dtype):
    """eps and sigma^2 of every pair of a batch of particle sets ([B, m] 0 = A, 1 = B)."""
    p = is_b[:, :, None] + is_b[:, None, :]
    eps = torch.tensor(md.KA_EPS, dtype=dtype, device=is_b.device)[p]
    sig = torch.tensor(md.KA_SIGMA, dtype=dtype, device=is_b.device)[p]
    return eps, sig * sig


def _melt(sets, seed, steps=160, dt=0.004, redraw=20):
    """Liquids of a batch of small boxes by a plain MD loop (all pairs, FP32):
    sets: (n_a, n_b, box, T).  Returns a list of float64 arrays [3, n], A first."""
    g = torch.Generator().manual_seed(seed)
    m = max(a + b for a, b, _, _ in sets)
    B = len(sets)
    x = torch.zeros(B, m, 3)
    is_b = torch.zeros(B, m, dtype=torch.int64)
    live = torch.zeros(B, m, dtype=torch.bool)
    for k, (a, b, L, _) in enumerate(sets):
        n = a + b
        s = math.ceil(n ** (1.0 / 3.0) - 1e-9)
        q = torch.randperm(s ** 3, generator=g)[:n]
        at = torch.stack([q % s, (q // s) % s, q // (s * s)], 1) + 0.5 + 0.1 * (torch.rand(n, 3, generator=g) - 0.5)
        x[k, :n] = at * (L / s)
        is_b[k, a:n] = 1
        live[k, :n] = True
    x, is_b, live = x.cuda(), is_b.cuda(), live.cuda()
    L = torch.tensor([s[2] for s in sets], device="cuda")[:, None, None]
    T = torch.tensor([s[3] for s in sets], device="cuda")[:, None, None]
    eps, sig2 = _pair_tables(is_b, torch.float32)
    both = live[:, :, None] & live[:, None, :] & ~torch.eye(m, dtype=torch.bool, device="cuda")[None]
    e48 = torch.where(both, 48.0 * eps, torch.zeros_like(eps))
    rc2 = 6.25 * sig2

    def force(x):
        d = [x[:, :, None, k] - x[:, None, :, k] for k in range(3)]
        d = [u - L * torch.round(u / L) for u in d]
        r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + 1e-6
        s6 = (sig2 / r2) ** 3
        f = torch.where(r2 < rc2, e48 * s6 * (s6 - 0.5) / r2, torch.zeros_like(r2)).clamp_(max=2000.0)
        return torch.stack([(f * u).sum(2) for u in d], 2)

    a = force(x)
    v = torch.zeros_like(x)
    for step in range(steps):
        if step % redraw == 0:
            v = (torch.randn(B, m, 3, generator=g).cuda() * torch.sqrt(T)) * live[:, :, None]
        v = v + 0.5 * dt * a
        x = x + dt * v
        a = force(x)
        v = v + 0.5 * dt * a
    x = torch.remainder(x.double(), L.double()).cpu().numpy()
    return [x[k, :sa + sb].T.copy() for k, (sa, sb, _, _) in enumerate(sets)]


def _inputs(case, seed):
    """Positions [3, n_total] and velocities [3, n_total] (numpy FP64, replicas
    one after the other, A before B), and the replicas."""
    reps = _replicas(case)
    tiles, sets = [], []
    for n, na, L, T in reps:
        k = max(1, math.ceil((n / 600.0) ** (1.0 / 3.0)))
        while k > 1 and L / k < 5.6:
            k -= 1
        tiles.append(k)
        sets.append((-(-na // k ** 3), -(-(n - na) // k ** 3), L / k, T))
    order = sorted(range(len(sets)), key=lambda r: sets[r][0] + sets[r][1])
    bases = [None] * len(sets)
    at = 0
    while at < len(order):  # batches of similar sizes
        group = order[at:at + 32]
        for r, p in zip(group, _melt([sets[r] for r in group], 1000 * seed + at)):
            bases[r] = p
        at += len(group)
    rng = np.random.default_rng(seed)
    pos, vel = [], []
    for (n, na, L, T), k, (a0, b0, L0, _), base in zip(reps, tiles, sets, bases):
        shift = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij")).reshape(3, 1, -1) * L0
        parts = []
        for sub, keep in ((base[:, :a0], na), (base[:, a0:], n - na)):
            full = (sub[:, :, None] + shift).reshape(3, -1)
            parts.append(full[:, rng.permutation(full.shape[1])[:keep]])
        p = np.mod(np.concatenate(parts, 1), L)
        p[p >= L] = 0.0
        v = rng.normal(0.0, math.sqrt(T), (3, n))
        v -= v.mean(1, keepdims=True)
        v *= math.sqrt(3.0 * n * T / np.sum(v * v))
        pos.append(p)
        vel.append(v)
    return np.concatenate(pos, 1), np.concatenate(vel, 1), reps


def _moved(case, seed, pos, L):
    """The displaced configuration of a `move` case: wrapped positions and image counters."""
    u = pos + np.random.default_rng(seed + 77).normal(0.0, 0.06, pos.shape)
    img = np.floor(u / L)
    p = u - img * L
    img[p >= L] += 1.0
    p[p >= L] = 0.0
    img[p < 0.0] -= 1.0
    p[p < 0.0] += L
    return p, img.astype(np.int32)


def prepare(case, seed):
    pos, vel, reps = _inputs(case, seed)
    s = md.System([(n, na, L, T, W.BASE_SEED + seed + 31 * r) for r, (n, na, L, T) in enumerate(reps)],
                  precision=case["precision"], dt=0.005, skin=case["skin"], positions=pos, velocities=vel)
    st = {"case": case, "sys": s}
    op, steps = case["op"], case["steps"]
    if op in ("nve", "bath", "nose") and case["graph"]:
        s.capture(steps, 0 if op == "nve" else 1, md.NVT_NOSE_HOOVER if op == "nose" else md.NVT_STOCHASTIC,
                  case["every"] or steps, 0.5)
    elif op == "move":
        s.msd_set_origin(0)
        p, img = _moved(case, seed, pos, reps[0][2])
        with torch.cuda.stream(s.stream):
            for k, u in zip(("x", "y", "z"), p):
                s.t[k].copy_(torch.from_numpy(np.ascontiguousarray(u)))
            s.img.copy_(torch.from_numpy(img))
        md.md_import(s.ctx)
    return st


def run(state):
    case, s = state["case"], state["sys"]
    op = case["op"]
    if op in ("nve", "bath", "nose"):
        if case["graph"]:
            s.launch()
        elif op == "nve":
            s.step_nve(case["steps"])
        elif op == "bath":
            s.step_nvt(case["steps"], md.NVT_STOCHASTIC, n_reassign=case["every"])
        else:
            s.step_nvt(case["steps"], md.NVT_NOSE_HOOVER, tau=0.5)
        return dict({k: s.t[k] for k in STATE}, img=s.img)
    if op == "forces":
        s.build_cells()
        pe_w = s.forces(energy=True)
        return {"pe_w": pe_w, "ax": s.t["ax"], "ay": s.t["ay"], "az": s.t["az"]}
    if op == "rdf":
        return {"hist": s.rdf(case["rmax"] / case["bins"], case["bins"])}
    return {"msd": s.msd(0), "hist": s.van_hove(0, 0.5 / case["bins"], case["bins"])}


# --------------------------------------------------------------- yardsticks
def _pairs(case, r=None):
    """Ordered pairs within the cutoffs (or within r) at uniform density."""
    tot = 0.0
    for n, na, L, _ in _replicas(case):
        V = L ** 3
        nb = n - na
        rr = [r] * 3 if r else [2.5 * s for s in md.KA_SIGMA]
        tot += sum(c * 4.0 / 3.0 * math.pi * q ** 3 for c, q in zip((na * na, 2 * na * nb, nb * nb), rr)) / V
    return tot


def work(case):
    n = sum(r[0] for r in _replicas(case))
    state = n * (9 * 8 + 12)
    op = case["op"]
    if op in ("nve", "bath", "nose"):
        return {"bytes": 2 * state, "flops": case["steps"] * (FLOP_PER_PAIR * _pairs(case) + 30 * n)}
    if op == "forces":
        return {"bytes": n * 48, "flops": (FLOP_PER_PAIR + 4) * _pairs(case)}
    if op == "rdf":
        return {"bytes": n * 24, "flops": 10 * _pairs(case, case["rmax"]) / 2}
    return {"bytes": n * (24 + 12 + 24) * 2, "flops": 16 * n}


# -------------------------------------------------- the same in 64-bit torch
class _Brute:
    """All-pairs forces of one replica in binary64 (torch, by blocks of rows)."""

    def __init__(self, n, na, L):
        self.n, self.L = n, L
        self.is_b = (torch.arange(n, device="cuda") >= na).to(torch.int64)
        self.eps = torch.tensor(md.KA_EPS, dtype=torch.float64, device="cuda")
        self.sig = torch.tensor(md.KA_SIGMA, dtype=torch.float64, device="cuda")

    def __call__(self, x, energy=False):
        n, L = self.n, self.L
        out, pe, w = torch.empty_like(x), 0.0, 0.0
        rows = max(1, 32_000_000 // n)
        for i in range(0, n, rows):
            d = x[:, i:i + rows, None] - x[:, None, :]
            d -= L * torch.round(d / L)
            r2 = (d * d).sum(0)
            p = self.is_b[i:i + rows, None] + self.is_b[None, :]
            s2 = (self.sig * self.sig)[p]
            on = (r2 < 6.25 * s2) & (r2 > 0.0)
            ir2 = torch.where(on, 1.0 / r2, torch.zeros_like(r2))
            s6 = (s2 * ir2) ** 3
            e = self.eps[p]
            f = 48.0 * e * s6 * (s6 - 0.5) * ir2
            for k in range(3):
                out[k, i:i + rows] = (f * d[k]).sum(1)
            if energy:
                c6 = 2.5 ** -6
                pe += float(torch.where(on, 4.0 * e * (s6 * s6 - s6 - (c6 * c6 - c6)), torch.zeros_like(e)).sum()) / 2
                w += float((f * r2).sum()) / 2
        return (out, pe, w) if energy else out


def exact(case, seed):
    """None for histograms (whole numbers), for the random draws of the bath,
    and where all pairs in binary64 would take too long."""
    op, dt = case["op"], 0.005
    if op in ("rdf", "bath"):
        return None
    reps = _replicas(case)
    passes = 1 + (case["steps"] if op != "forces" else 0)
    if op != "move" and passes * sum(r[0] ** 2 + 4e6 for r in reps) > 6e10:
        return None
    pos, vel, reps = _inputs(case, seed)
    if op == "move":
        n, na, L, _ = reps[0]
        p, img = _moved(case, seed, pos, L)
        d2 = ((p + img * L - pos) ** 2).sum(0)
        return {"msd": np.array([[d2[:na].mean(), d2[na:].mean()]]), "hist": None}
    if op == "forces":
        n, na, L, _ = reps[0]
        a, pe, w = _Brute(n, na, L)(torch.from_numpy(pos).cuda(), True)
        return {"pe_w": np.array([[pe, w]]), "ax": a[0], "ay": a[1], "az": a[2]}
    got, at = [], 0
    for n, na, L, T in reps:
        force = _Brute(n, na, L)
        x = torch.from_numpy(pos[:, at:at + n].copy()).cuda()
        v = torch.from_numpy(vel[:, at:at + n].copy()).cuda()
        at += n
        img = torch.zeros(3, n, dtype=torch.float64, device="cuda")
        a = force(x)
        xi, Q, X = 0.0, 3.0 * n * T * 0.25, 3.0 * n
        for _ in range(case["steps"]):
            G = (float((v * v).sum()) - X * T) / Q if op == "nose" else 0.0
            xia = xi + G * dt
            c = 0.5 * dt * (1.0 - 0.5 * dt * xia) if op == "nose" else 0.5 * dt
            x = x + dt * (v + 0.5 * dt * (a - xi * v))
            v = v + c * (a - (xi + xia) * v)
            k = torch.floor(x / L)
            x, img = x - k * L, img + k
            a = force(x)
            v = v + c * a
            if op == "nose":
                xi = xi + 0.5 * dt * (G + (float((v * v).sum()) - X * T) / Q)
        got.append(torch.cat([x, v, a], 0))
    got = torch.cat(got, 1)
    return dict({k: got[i] for i, k in enumerate(STATE)}, img=None)
