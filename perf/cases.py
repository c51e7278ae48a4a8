"""The framework's work, as cases that can be timed: what a user has it do, over the sizes,
precisions and options in use.

Four kinds of pass, each through the package's public entry points:

  sweep    Lattice.sweep: Monte Carlo and over-relaxation sweeps of one resident lattice
  pt       one block of a parallel-tempering run: PTRunner.run_cycle over a batch of chains
           (sweeps, a replica exchange, the overlaps of the replicas)
  serve    Server.run on a closed trace of simulation requests of mixed size
  observe  the measurements of two replicas of one lattice: tensor overlap, Fourier
           overlaps, recomputed energy

Inputs are made from the seed alone.  Single lattices start from a quenched state (a few
noisy alignments of random spins to their local fields), which accepts and rejects as a
cold run does; chains and requests start, as a user's do, from the library's own random
state and the seeds they name.  ``exact`` computes a pass in binary64 with plain torch.
"""
import math
import random

import torch

import paper_1006_2566_amd as hsg
from paper_1006_2566_amd import batch as hb
from paper_1006_2566_amd import serve as sv

DTYPES = {"f32": torch.float32, "f64": torch.float64}
TWO32 = 0xFFFFFFFF


def _sweep(name, L, n_sweeps, dtype="f32", k=4, n_or=1, T=0.3, renorm=10, heat_bath=False):
    return {"name": name, "kind": "sweep", "L": L, "dtype": dtype, "k": k, "n_or": n_or, "T": T,
            "renorm": renorm, "heat_bath": heat_bath, "n_sweeps": n_sweeps}


def listed():
    return [
        # validation runs and finite-size series begin here: launches and latency alone
        _sweep("sweep_L8", 8, 10, T=0.5),
        # a small production lattice, heat bath with over-relaxation between measurements
        _sweep("heat_bath_L24", 24, 4, k=1, n_or=2, T=0.2, heat_bath=True),
        # the single-lattice workload of the tests (L = 64, T = 0.2 .. 1, k = 1, 4, 8)
        _sweep("sweep_L64", 64, 4, T=0.5),
        # the paper's own benchmark: over-relaxation alone, L = 128, binary32
        _sweep("over_relax_L128", 128, 20, k=0, n_or=1, T=1.0, renorm=0),
        # a size that no tile divides, in binary64, single hits
        _sweep("sweep_L100_f64", 100, 2, dtype="f64", k=1, n_or=1, T=0.4),
        # ... and one in binary32, with two over-relaxation phases to each heat-bath phase
        _sweep("heat_bath_L150", 150, 2, k=1, n_or=2, T=0.3, heat_bath=True),
        # the headline: L = 256, binary32, k = 4 and one over-relaxation phase
        _sweep("sweep_L256", 256, 4),
        # the large-lattice configuration: k = 4 and two over-relaxation phases
        _sweep("sweep_L512", 512, 2, n_or=2),
        # one disorder sample at L = 32: 2 replicas of 24 temperatures
        {"name": "pt_one_sample", "kind": "pt", "samples": 1, "Ls": "32", "temps": 24, "k": 4,
         "sweeps": 10},
        # the batched workload: 256 samples of mixed size, 12288 chains
        {"name": "pt_256_samples", "kind": "pt", "samples": 256, "Ls": "16,24,32,48", "temps": 24,
         "k": 4, "sweeps": 10},
        # the served stream's sizes and hits, short requests
        {"name": "serve_48", "kind": "serve", "requests": 48, "Ls": "8,16,32,64,96",
         "min_sweeps": 32, "max_sweeps": 128},
        # one measurement of two replicas of the headline lattice
        {"name": "observe_L256", "kind": "observe", "L": 256, "dtype": "f32"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _even(rng, lo, hi):
    return max(lo, min(hi, 2 * _log_int(rng, lo / 2, hi / 2)))


def draw(rng):
    kind = rng.choices(["sweep", "pt", "serve", "observe"], weights=[12, 3, 2, 3])[0]
    if kind == "sweep":
        L = _even(rng, 8, 384)
        heat_bath = rng.random() < 0.25
        k = 1 if heat_bath else rng.choice([0, 1, 1, 2, 4, 4, 8])
        n_or = rng.randint(1 if k == 0 else 0, 3)
        c = _sweep("", L, rng.randint(1, 10 if L < 128 else 4), dtype=rng.choice(["f32"] * 3 + ["f64"]),
                   k=k, n_or=n_or, T=round(rng.uniform(0.1, 1.0), 3),
                   renorm=rng.choice([0, 1, 10]), heat_bath=heat_bath)
        del c["name"]
        return c
    if kind == "pt":
        Ls = rng.choice(["8,16", "16,24,32,48", "12,20", "16,32", "10,18,36", "24", "40"])
        return {"kind": "pt", "samples": _log_int(rng, 1, 48), "Ls": Ls,
                "temps": rng.randint(8, 32), "k": rng.choice([1, 4]), "sweeps": rng.randint(2, 12)}
    if kind == "serve":
        lo = _log_int(rng, 8, 64)
        return {"kind": "serve", "requests": _log_int(rng, 4, 64),
                "Ls": rng.choice(["8,16,32,64,96", "8,16,32", "10,24,48", "32,64"]),
                "min_sweeps": lo, "max_sweeps": lo * 4}
    return {"kind": "observe", "L": _even(rng, 16, 320), "dtype": rng.choice(["f32", "f32", "f64"])}


# ------------------------------------------------------------------ inputs in plain torch


def _field(s, J, L):
    """Local field of every site, s and J of shape (3, L, L, L) indexed [a, z, y, x]."""
    h = torch.zeros_like(s)
    for d, dim in enumerate((3, 2, 1)):  # x, y, z bonds
        h += J[d] * torch.roll(s, -1, dim)
        h += torch.roll(J[d] * s, 1, dim)
    return h


def _colour_mask(L, colour, device):
    i = torch.arange(L, device=device)
    return ((i[:, None, None] + i[None, :, None] + i[None, None, :]) & 1) == colour


def _unit(v):
    return v / v.square().sum(0, keepdim=True).sqrt()


def _state(L, dtype, seed, device, T=0.3):
    """Quenched spins and Gaussian couplings, shape (3, L, L, L) each."""
    g = torch.Generator(device=device).manual_seed(seed)
    J = torch.randn(3, L, L, L, generator=g, device=device, dtype=dtype)
    s = _unit(torch.randn(3, L, L, L, generator=g, device=device, dtype=dtype))
    for _ in range(4):
        for colour in (0, 1):
            t = _unit(_field(s, J, L).add_(torch.randn(s.shape, generator=g, device=device, dtype=dtype), alpha=2 * T))
            s = torch.where(_colour_mask(L, colour, device), t, s)
            del t
    return s, J


def _lattice(case, seed, state_seed=None):
    L, dtype = case["L"], DTYPES[case["dtype"]]
    lat = hsg.Lattice(L, dtype, seed=seed, device="cuda", init=None)
    s, J = _state(L, dtype, seed if state_seed is None else state_seed, "cuda")
    lat.load(s.reshape(3, -1), J.reshape(3, -1))
    return lat


def _second_replica(case, seed):
    L, dtype = case["L"], DTYPES[case["dtype"]]
    _, J = _state(L, dtype, seed, "cuda")
    s, _ = _state(L, dtype, seed + 7919, "cuda")
    lat = hsg.Lattice(L, dtype, seed=seed + 1, device="cuda", init=None)
    lat.load(s.reshape(3, -1), J.reshape(3, -1))
    return lat


# ------------------------------------------------------------------------- the passes


def prepare(case, seed):
    kind = case["kind"]
    if kind == "sweep":
        return {"case": case, "lat": _lattice(case, seed)}
    if kind == "pt":
        specs, ladders, betas, pairs = hb.pt_workload(
            n_samples=case["samples"], Ls=tuple(int(v) for v in case["Ls"].split(",")),
            n_temps=case["temps"], k=case["k"])
        g = random.Random(seed)  # the sizes are the workload's, the disorder and the draws the seed's
        J_seeds = [g.getrandbits(63) for _ in range(case["samples"])]
        for c in specs:
            c.seed, c.J_seed = g.getrandbits(63), J_seeds[c.J_group]
        b = hb.Batch(specs)
        pt = hb.Tempering(b, ladders, betas, seed=seed)
        return {"case": case, "batch": b, "pt": pt,
                "runner": hb.PTRunner(b, pt, pairs, sweeps_per_exchange=case["sweeps"],
                                      exchanges_per_measure=1)}
    if kind == "serve":
        trace = sv.poisson_trace(n=case["requests"], seed=seed,
                                 Ls=tuple(int(v) for v in case["Ls"].split(",")),
                                 sweep_range=(case["min_sweeps"], case["max_sweeps"]))
        for r in trace:
            r.seed += 10000 * (seed % 1000003)
        return {"case": case, "trace": trace, "server": sv.Server(hbm_budget=2 << 30, n_slots=128)}
    return {"case": case, "a": _lattice(case, seed), "b": _second_replica(case, seed)}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "sweep":
        lat = state["lat"]
        lat.sweep(T=case["T"], k=case["k"], n_or=case["n_or"], renorm_every=case["renorm"],
                  n_sweeps=case["n_sweeps"], heat_bath=case["heat_bath"])
        return {"spins": lat.spins, "E": lat.energy()}
    if kind == "pt":
        state["runner"].run_cycle()
        return {"spins": state["batch"].spins, "E": state["batch"].E,
                "slots": state["pt"].chain_at_slot, "beta": state["batch"].beta,
                "q": state["runner"].q}
    if kind == "serve":
        res = sorted(state["server"].run(state["trace"], realtime=False), key=lambda r: r.rid)
        return {"E": torch.tensor([r.E for r in res], dtype=torch.float64),
                "m": torch.tensor([[float(v) for v in r.m] for r in res], dtype=torch.float64),
                "sweeps": torch.tensor([r.sweeps_done for r in res])}
    a, b = state["a"], state["b"]
    return {"overlap": a.overlap(b), "fourier": a.overlap_fourier(b),
            "E": a.energy(recompute=True)}


def _pt_sizes(case):
    """Mean number of sites of a chain, and the number of chains."""
    Ls = [int(v) for v in case["Ls"].split(",")]
    return sum(L ** 3 for L in Ls) / len(Ls), case["samples"] * 2 * case["temps"]


def work(case):
    """Bytes: the state read once and the spins written once per call.  Flops: the field
    (36 per site and phase), 24 per over-relaxation update, 60 per Metropolis hit or
    heat-bath draw; the integer work of the generator is not counted."""
    kind = case["kind"]
    if kind == "sweep":
        N, es = case["L"] ** 3, 4 if case["dtype"] == "f32" else 8
        draws = 1 if case["heat_bath"] else case["k"]
        per = (36 + 60 * draws if draws else 0) + 60 * case["n_or"]
        return {"bytes": 9 * N * es, "flops": float(N) * case["n_sweeps"] * per}
    if kind == "pt":
        N, chains = _pt_sizes(case)
        return {"bytes": 4 * N * (6 * chains + 3 * case["samples"]),
                "flops": N * chains * (case["sweeps"] * (36 + 60 * case["k"]) + 24)}
    if kind == "serve":
        Ls = [int(v) for v in case["Ls"].split(",")]
        N = sum(L ** 3 for L in Ls) / len(Ls) * case["requests"]
        mean = (case["max_sweeps"] - case["min_sweeps"]) / math.log(case["max_sweeps"] / case["min_sweeps"])
        return {"bytes": 36 * N, "flops": N * mean * (36 + 60 * 2.5)}
    N, es = case["L"] ** 3, 4 if case["dtype"] == "f32" else 8
    return {"bytes": 9 * N * es, "flops": N * (36 + 30 + 90)}


# ---------------------------------------------------------------- the same in binary64


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 (Salmon et al., 2011) on int64 tensors holding 32-bit words."""
    k0, k1 = seed & TWO32, (seed >> 32) & TWO32
    for _ in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c2 = ((b >> 32) & TWO32) ^ c1 ^ k0, ((a >> 32) & TWO32) ^ c3 ^ k1
        c1, c3 = b & TWO32, a & TWO32
        k0, k1 = (k0 + 0x9E3779B9) & TWO32, (k1 + 0xBB67AE85) & TWO32
    return c0, c1, c2, c3


def _uniforms(site, sweep, phase, first, count, tag, seed):
    """Uniforms first .. first + count - 1 of every site's stream in one phase."""
    out = []
    for block in range(first // 4, (first + count - 1) // 4 + 1):
        c0, c2, c3 = (torch.full_like(site, v) for v in (sweep, (phase << 16) | block, tag))
        out += [(2 * (w >> 9) + 1).double() * 2.0 ** -24 for w in _philox(c0, site, c2, c3, seed)]
    return out[first % 4:first % 4 + count]


def _point(z, u):
    rho = (1 - z * z).clamp_min(0).sqrt()
    return torch.stack([rho * torch.cos(2 * math.pi * u), rho * torch.sin(2 * math.pi * u), z])


def _dot(a, b):
    return (a * b).sum(0)


def _heat_bath_spin(h, beta, u0, u1):
    """Cosine to the field by inversion, azimuth in the branch-free tangent frame of
    Duff et al. (JCGT 2017)."""
    hn = _dot(h, h).sqrt()
    a = beta * hn
    wq = (1 - u0) * -torch.expm1(-2 * a)
    c = 1 + torch.where(wq <= 0.5, torch.log1p(-wq), torch.log(u0 + (1 - u0) * torch.exp(-2 * a))) / a
    c = c.clamp(-1, 1)
    p = _point(c, u1)
    n = h / hn
    sgn = torch.where(n[2] >= 0, 1.0, -1.0).double()
    ia = -1 / (sgn + n[2])
    b = n[0] * n[1] * ia
    e1 = torch.stack([1 + sgn * n[0] * n[0] * ia, sgn * b, -sgn * n[0]])
    e2 = torch.stack([b, sgn + n[1] * n[1] * ia, -n[1]])
    return c * n + p[0] * e1 + p[1] * e2


def _exact_sweep(case, seed, device):
    L = case["L"]
    s, J = (v.double() for v in _state(L, DTYPES[case["dtype"]], seed, device))
    site = torch.arange(L ** 3, device=device).reshape(L, L, L)
    beta = 1.0 / case["T"]
    masks = [_colour_mask(L, c, device) for c in (0, 1)]
    for n in range(case["n_sweeps"]):
        for phase in range(0 if case["k"] else 1, case["n_or"] + 1):
            for colour in (0, 1):
                h = _field(s, J, L)
                if phase:
                    t = 2 * _dot(s, h) / _dot(h, h) * h - s
                elif case["heat_bath"]:
                    u = _uniforms(site, n, 0, 2 * (case["k"] - 1), 2, 5, seed)
                    t = _heat_bath_spin(h, beta, *u)
                else:
                    t = s.clone()
                    for j in range(case["k"]):
                        u = _uniforms(site, n, 0, 3 * j, 3, 0, seed)
                        trial = _point(2 * u[0] - 1, u[1])
                        dE = _dot(t, h) - _dot(trial, h)
                        take = (dE <= 0) | (u[2] < torch.exp(-beta * dE))
                        t = torch.where(take, trial, t)
                s = torch.where(masks[colour], t, s)
        if case["renorm"] and (n + 1) % case["renorm"] == 0:
            s = _unit(s)
    E = -0.5 * _dot(s, _field(s, J, L)).sum()
    return {"spins": _colour_split(s, L), "E": E.reshape(1)}


def _colour_split(v, L):
    """Six planes of N/2 values, plane 3c + a: component a of the colour-c sites in
    (z, y, x/2) order."""
    planes = []
    for c in (0, 1):
        m = _colour_mask(L, c, v.device)
        planes += [v[a][m] for a in range(3)]
    return torch.cat(planes)


def _exact_observe(case, seed, device):
    L, dtype = case["L"], DTYPES[case["dtype"]]
    N = L ** 3
    a, J = (v.double() for v in _state(L, dtype, seed, device))
    b = _state(L, dtype, seed + 7919, device)[0].double()
    q = torch.stack([a[m] * b[n] for m in range(3) for n in range(3)]) / N
    ma, mb = (v.reshape(3, -1).sum(1) / N for v in (a, b))
    q0 = q.reshape(9, -1).sum(1)
    ang = 2 * math.pi * torch.arange(L, device=device).double() / L
    parts = []
    for dims in ((1, 2), (1, 3), (2, 3)):  # sums over the axes other than x, y, z
        line = q.sum(dims)
        parts += [(line * torch.cos(ang)).sum(1), (line * torch.sin(ang)).sum(1)]
    qk = torch.cat(parts)
    fourier = torch.cat([q0, qk, q0.square().sum().reshape(1), qk.square().sum().reshape(1) / 3])
    E = -0.5 * _dot(a, _field(a, J, L)).sum()
    return {"overlap": torch.cat([q0, ma, mb]), "fourier": fourier, "E": E.reshape(1)}


def exact(case, seed):
    """Binary64 values of run() on the case's inputs; None for long runs (a decision taken
    the other way travels through all that follows) and for many lattices at once."""
    device = "cuda" if torch.cuda.is_available() else "cpu"
    if case["kind"] == "observe":
        return _exact_observe(case, seed, device)
    if case["kind"] == "sweep" and case["n_sweeps"] <= 4 and case["L"] <= 256:
        return _exact_sweep(case, seed, device)
    return None
