"""The work that users of this library have it do, as timed cases.

Each kind is one use of the library through its public entry points: a single
chain, a table of diagonal correlations, a sweep of a few chains, a batched
(q, J) scan, exact sampling, recorded trajectories and their likelihood, one
ascent step of a fit, and replica-coded chains.  `listed()` gives one or two
sizes of each, from the smallest calls to the largest; `draw(rng)` gives
further sizes of the same ranges.  A pass that runs chains starts from a fresh
initial lattice, as a program that starts a chain does, so that it can be
repeated on the same state.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1908_07341_amd as sd
from paper_1908_07341_amd import autograd, inputs

LAYOUTS = {"int8": sd.SD_I8, "p32": sd.SD_P32, "p64": sd.SD_P64}
STARTS = {"up": sd.SD_INIT_UP, "down": sd.SD_INIT_DOWN, "random": sd.SD_INIT_RANDOM}

# 32-bit integer operations of one spin update: its share of the counter-based
# uniforms (4 calls per 64 sites, one more per 256 sites, 40 operations each)
# and of the bit-sliced comparison (8 planes of 3 operations per 32 sites).
OPS_PER_UPDATE = (4.0 / 64.0 + 1.0 / 256.0) * 40.0 + 8 * 3 / 32.0


def listed():
    return [
        # 10^4 recorded steps of a 64^2 int8 chain from all +1 is the smallest
        # run that the benchmark's oracle plan lists; a tenth of it here
        {"name": "chain_64_int8", "kind": "chain", "L": 64, "layout": "int8", "start": "up", "J": 0.4, "q": 0.6,
         "steps": 1000, "obs_every": 1},
        # int8 spins on an odd lattice: the general layout, any L
        {"name": "chain_333_int8", "kind": "chain", "L": 333, "layout": "int8", "start": "random", "J": 0.5,
         "q": 0.8, "steps": 200, "obs_every": 10},
        # the headline chain: 16384^2 packed, a record every 10 steps
        {"name": "chain_16384_packed", "kind": "chain", "L": 16384, "layout": "p64", "start": "random", "J": 0.5,
         "q": 0.5, "steps": 20, "obs_every": 10},
        # Table 1's time averages on the 32^2 box: 5 steps between measurements
        # of the diagonal correlations, many small calls
        {"name": "table_32", "kind": "table", "L": 32, "layout": "p32", "J": 0.66, "q": 1.0, "every": 5,
         "measurements": 20, "lmax": 16},
        # the five-point sweep: 1024^2 int8, a record every step, D(r) every
        # 100 steps
        {"name": "sweep_1024", "kind": "sweep", "L": 1024, "layout": "int8", "chains": 5, "steps": 100,
         "obs_every": 1, "rmax": 512},
        # the (q, J) scan of 4096 chains of 128^2, 256^2 and 512^2, a record
        # every step (5000 steps in the benchmark)
        {"name": "scan_4096", "kind": "scan", "n_q": 64, "n_J": 64, "sizes": "128,256,512", "layout": "p64",
         "steps": 100, "obs_every": 1, "moments": False},
        # the critical-curve scan: 200^2 from all -1, moments of the
        # magnetisation (80 x 80 grid, 3e5 steps in the benchmark)
        {"name": "critical_200", "kind": "scan", "n_q": 40, "n_J": 40, "sizes": "200", "layout": "p64",
         "steps": 200, "obs_every": 1, "moments": True},
        # exact samples of the 32^2 box by coupling from the past
        {"name": "exact_samples_32", "kind": "exact_samples", "L": 32, "samples": 512, "J": 0.38, "q": 2.5,
         "T0": 16, "T_max": 1 << 20},
        # recording the trajectories of a fit (2000 steps in the benchmark)
        {"name": "trajectories_256", "kind": "trajectories", "L": 256, "chains": 256, "J": 0.45, "q": 0.7,
         "steps": 100},
        # the 12 counts of recorded trajectories, larger than the caches
        {"name": "counts_256", "kind": "counts", "L": 256, "chains": 256, "J": 0.45, "q": 0.7, "steps": 500,
         "paired": False},
        # one step of the gradient ascent: LL and its gradient from the counts,
        # the smallest calls of all
        {"name": "ascent_step", "kind": "ascent", "sites": 67108864000, "J": 0.45, "q": 0.7, "at_J": 0.2,
         "at_q": 0.2, "paired": False},
        # 64 replica-coded chains sharing one stream, and their observables
        {"name": "replicas_2048", "kind": "replicas", "L": 2048, "q": 1.0, "steps": 8},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _coupling(rng):
    return round(rng.uniform(0.1, 1.0), 3), round(rng.uniform(0.1, 2.0), 3)


def _draw_chain(rng):
    layout = rng.choice(["int8", "int8", "p64", "p64", "p32"])
    if layout == "int8":
        L = _log_int(rng, 17, 2048)
    elif layout == "p64":
        L = 8 * _log_int(rng, 2, 2048)
    else:
        L = 32 * _log_int(rng, 1, 256)
    J, q = _coupling(rng)
    budget = 2e8 if layout == "int8" else 5e9
    steps = max(2, min(_log_int(rng, 100, 1000), int(budget / (2 * L * L))))
    return {"kind": "chain", "L": L, "layout": layout, "start": rng.choice(list(STARTS)), "J": J, "q": q,
            "steps": steps, "obs_every": rng.choice([0, 1, 2, 10])}


def _draw_table(rng):
    layout = rng.choice(["p32", "p64", "int8"])
    L = {"p32": 32 * rng.randint(1, 8), "p64": 8 * rng.randint(2, 32), "int8": rng.randint(16, 256)}[layout]
    J, q = _coupling(rng)
    return {"kind": "table", "L": L, "layout": layout, "J": J, "q": q, "every": rng.randint(1, 10),
            "measurements": rng.randint(5, 30), "lmax": rng.randint(1, L // 2)}


def _draw_sweep(rng):
    layout = rng.choice(["int8", "p64"])
    L = 64 * _log_int(rng, 1, 32)
    steps = max(3, min(100, int(2e9 / (2 * L * L * 5))))
    return {"kind": "sweep", "L": L, "layout": layout, "chains": rng.randint(1, 8), "steps": steps,
            "obs_every": rng.choice([1, 1, 5, 10]) if steps >= 10 else 1, "rmax": rng.randint(1, L // 2)}


def _draw_scan(rng):
    moments = rng.random() < 0.5
    if rng.random() < 0.5:
        sizes = sorted(rng.sample([64, 128, 192, 256, 320, 384, 512], rng.randint(1, 3)))
    else:
        sizes = [8 * rng.choice([k for k in range(4, 50) if k % 8])]
    n_q, n_J = rng.randint(4, 64), rng.randint(4, 64)
    layout = "p64" if len(sizes) == 1 and sizes[0] % 64 else rng.choice(["p64", "p64", "int8"])
    updates = 2.0 * n_q * n_J * sum(s * s for s in sizes) / len(sizes)
    steps = max(5, min(200, int(3e10 / updates)))
    return {"kind": "scan", "n_q": n_q, "n_J": n_J, "sizes": ",".join(map(str, sizes)), "layout": layout,
            "steps": steps, "obs_every": 1 if moments else rng.choice([1, 1, 5]), "moments": moments}


def _draw_exact_samples(rng):
    return {"kind": "exact_samples", "L": 8 * rng.randint(1, 8), "samples": _log_int(rng, 16, 512),
            "J": round(rng.uniform(0.1, 0.36), 3), "q": round(rng.uniform(0.3, 2.0), 3), "T0": 16, "T_max": 1 << 14}


def _draw_trajectories(rng):
    L = 8 * _log_int(rng, 4, 64)
    chains = _log_int(rng, 4, 256)
    steps = max(2, min(200, int(256 * 256 * 256 * 100 / (L * L * chains))))
    J, q = _coupling(rng)
    return {"kind": "trajectories", "L": L, "chains": chains, "J": J, "q": q, "steps": steps}


def _draw_counts(rng):
    L = 64 * _log_int(rng, 1, 12)
    chains = _log_int(rng, 4, 256)
    steps = max(4, min(600, int(256 * 256 * 256 * 400 / (L * L * chains))))
    J, q = _coupling(rng)
    return {"kind": "counts", "L": L, "chains": chains, "J": J, "q": q, "steps": steps,
            "paired": rng.random() < 0.5}


def _draw_ascent(rng):
    J, q = _coupling(rng)
    at_J, at_q = _coupling(rng)
    return {"kind": "ascent", "sites": _log_int(rng, 10 ** 5, 7 * 10 ** 10), "J": J, "q": q, "at_J": at_J,
            "at_q": at_q, "paired": rng.random() < 0.5}


def _draw_replicas(rng):
    L = 8 * _log_int(rng, 4, 256)
    steps = max(1, min(rng.randint(4, 40), int(8 * 2048 * 2048 / (L * L))))
    return {"kind": "replicas", "L": L, "q": round(rng.uniform(0.3, 2.0), 3), "steps": steps}


_DRAW = [_draw_chain, _draw_chain, _draw_table, _draw_sweep, _draw_scan, _draw_exact_samples, _draw_trajectories,
         _draw_counts, _draw_ascent, _draw_replicas]


def draw(rng):
    return rng.choice(_DRAW)(rng)


def _scan_table(case):
    sizes = [int(s) for s in case["sizes"].split(",")]
    return inputs.scan_table(n_q=case["n_q"], n_J=case["n_J"], sizes=sizes)


def _ascent_counts(case, seed):
    """The 12 counts that `sites` site draws at the generating (J, q) leave:
    classes as a chain near equilibrium has them, every draw from its field."""
    rng = np.random.default_rng(seed)
    cls = rng.multinomial(case["sites"], [0.28, 0.05, 0.17, 0.17, 0.05, 0.28])
    counts = np.zeros(12, dtype=np.int64)
    for idx in range(6):
        h = case["J"] * (2 * (idx >> 1) - 2) + case["q"] * (2 * (idx & 1) - 1)
        plus = rng.binomial(cls[idx], 1.0 / (1.0 + math.exp(-2.0 * h)))
        counts[2 * idx], counts[2 * idx + 1] = cls[idx] - plus, plus
    return counts


def _ascent_stats(case, seed):
    c = _ascent_counts(case, seed)
    if not case["paired"]:
        return c
    out = np.zeros(6, dtype=np.int64)
    for j in range(3):
        k = 5 - j
        out[j] = c[2 * j] + c[2 * j + 1] + c[2 * k] + c[2 * k + 1]
        out[3 + j] = c[2 * j + 1] + c[2 * k]
    return out


def _starts(n, L, seed):
    start = torch.empty((n, L * L // 64), dtype=torch.int64, device="cuda")
    for a in range(n):
        sd.sd_init(start[a], L, sd.SD_P64, sd.SD_INIT_RANDOM, 0.5, seed, a)
    return start


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "seed": seed}
    dev = "cuda"
    if kind in ("chain", "table"):
        lay = LAYOUTS[case["layout"]]
        s["sigma"], s["tau"] = sd.new_lattice(case["L"], lay), sd.new_lattice(case["L"], lay)
        if kind == "chain":
            n_rec = case["steps"] // case["obs_every"] if case["obs_every"] else 0
            s["obs"] = torch.empty((n_rec, 3), dtype=torch.int64, device=dev) if n_rec else None
        else:
            s["out"] = torch.empty((case["measurements"], 2, case["lmax"] + 1), dtype=torch.int64, device=dev)
    elif kind == "sweep":
        lay, n = LAYOUTS[case["layout"]], case["chains"]
        s["sigma"] = [sd.new_lattice(case["L"], lay) for _ in range(n)]
        s["tau"] = [sd.new_lattice(case["L"], lay) for _ in range(n)]
        s["points"] = [0.2 * (1 + a % 5) for a in range(n)]
        s["obs"] = torch.empty((n, case["steps"] // case["obs_every"], 3), dtype=torch.int64, device=dev)
        s["D"] = torch.empty((n, case["rmax"] + 1), dtype=torch.int64, device=dev)
    elif kind == "scan":
        q, J, L = _scan_table(case)
        s["plan"] = sd.sd_batch_plan_create(J, q, L, list(range(len(L))), layout=LAYOUTS[case["layout"]], seed=seed,
                                            k_steps=case["steps"], obs_every=case["obs_every"],
                                            flags=sd.SD_FLAG_MOMENTS if case["moments"] else 0)
        # zeros: the plan pads its lattices, and the whole buffer is the output
        s["lattices"] = torch.zeros(sd.sd_batch_lattice_bytes(s["plan"]), dtype=torch.uint8, device=dev)
        s["traces"] = torch.zeros(sd.sd_batch_trace_len(s["plan"]), dtype=torch.int64, device=dev)
    elif kind == "exact_samples":
        nb = sd.sd_lattice_bytes(case["L"], sd.SD_P64)
        s["samples"] = torch.empty((case["samples"], nb), dtype=torch.uint8, device=dev)
        s["work"] = torch.empty(4 * case["samples"] * nb, dtype=torch.uint8, device=dev)
    elif kind in ("trajectories", "counts"):
        L, n, k = case["L"], case["chains"], case["steps"]
        s["start"] = _starts(n, L, seed)
        s["traj"] = torch.empty((n, 2 * k + 1, L * L // 64), dtype=torch.int64, device=dev)
        if kind == "counts":
            sd.sd_trajectories(s["start"], s["traj"], n, L, sd.SD_P64, case["J"], case["q"], seed, 0, 0, k)
    elif kind == "ascent":
        s["stats"] = torch.from_numpy(_ascent_stats(case, seed)).to(dev)
        s["Jq"] = torch.tensor([case["at_J"], case["at_q"]], dtype=torch.float32, device=dev, requires_grad=True)
    elif kind == "replicas":
        L = case["L"]
        g = torch.Generator(device=dev).manual_seed(seed)
        s["start"] = torch.randint(-2 ** 63, 2 ** 63 - 1, (L * L,), dtype=torch.int64, device=dev, generator=g)
        s["sigma"], s["tau"] = torch.empty_like(s["start"]), torch.empty_like(s["start"])
        s["J"], s["q"] = [1.5 * k / 63 for k in range(64)], [case["q"]] * 64
        s["out"] = torch.empty((64, 3), dtype=torch.int64, device=dev)
    return s


def run(s):
    case, seed = s["case"], s["seed"]
    kind = case["kind"]
    if kind == "chain":
        L, lay = case["L"], LAYOUTS[case["layout"]]
        sd.sd_init(s["sigma"], L, lay, STARTS[case["start"]], 0.5, seed, 0)
        sd.sd_run(s["sigma"], s["tau"], L, lay, case["J"], case["q"], seed, 0, 0, case["steps"], s["obs"],
                  case["obs_every"])
        return {"sigma": s["sigma"], "tau": s["tau"], "obs": s["obs"]} if s["obs"] is not None else \
            {"sigma": s["sigma"], "tau": s["tau"]}
    if kind == "table":
        L, lay = case["L"], LAYOUTS[case["layout"]]
        sd.sd_init(s["sigma"], L, lay, sd.SD_INIT_RANDOM, 0.5, seed, 0)
        for m in range(case["measurements"]):
            sd.sd_run(s["sigma"], s["tau"], L, lay, case["J"], case["q"], seed, 0, m * case["every"], case["every"],
                      None, 0)
            sd.sd_corr_diag(s["sigma"], L, lay, case["lmax"], s["out"][m])
        return {"sigma": s["sigma"], "out": s["out"]}
    if kind == "sweep":
        L, lay, n = case["L"], LAYOUTS[case["layout"]], case["chains"]
        for a in range(n):
            sd.sd_init(s["sigma"][a], L, lay, sd.SD_INIT_RANDOM, 0.5, seed, a)
        sd.sd_run_many(s["sigma"], s["tau"], L, lay, s["points"], s["points"], seed, list(range(n)), 0,
                       case["steps"], s["obs"], case["obs_every"])
        sd.sd_corr_row_many(s["sigma"], L, lay, case["rmax"], s["D"])
        return {"sigma": s["sigma"], "tau": s["tau"], "obs": s["obs"], "D": s["D"]}
    if kind == "scan":
        sd.sd_batch_init(s["plan"], s["lattices"], sd.SD_INIT_DOWN if case["moments"] else sd.SD_INIT_RANDOM, 0.5)
        sd.sd_batch_run(s["plan"], s["lattices"], s["traces"], 0)
        return {"lattices": s["lattices"], "traces": s["traces"]}
    if kind == "exact_samples":
        T = sd.sd_propp_wilson(s["samples"], s["work"], case["samples"], case["L"], case["J"], case["q"], seed, 0,
                               1 << 28, case["T0"], case["T_max"])
        return {"samples": s["samples"], "T": np.array(T, dtype=np.int64)}
    if kind == "trajectories":
        sd.sd_trajectories(s["start"], s["traj"], case["chains"], case["L"], sd.SD_P64, case["J"], case["q"], seed,
                           0, 0, case["steps"])
        return s["traj"]
    if kind == "counts":
        f = autograd.loglik_stats if case["paired"] else autograd.loglik_counts
        return f(s["traj"], case["chains"], 2 * case["steps"] + 1, case["L"])
    if kind == "ascent":
        ll = autograd.loglik(s["Jq"], s["stats"])
        (grad,) = torch.autograd.grad(ll, s["Jq"])
        return {"ll": ll.detach(), "grad": grad}
    if kind == "replicas":
        s["sigma"].copy_(s["start"])
        sd.sd_replica_run(s["sigma"], s["tau"], case["L"], s["J"], s["q"], seed, 0, 0, case["steps"])
        sd.sd_replica_observe(s["sigma"], s["tau"], case["L"], s["out"])
        return {"sigma": s["sigma"], "tau": s["tau"], "out": s["out"]}
    raise ValueError(kind)


def work(case):
    kind = case["kind"]
    if kind == "ascent":
        return {"bytes": 8 * (6 if case["paired"] else 12) + 8 + 12, "flops": 2000}
    if kind == "scan":
        _, _, sizes = _scan_table(case)
        sites = float((sizes.astype(np.int64) ** 2).sum())
        per_site = 1.0 if case["layout"] == "int8" else 0.125
        rec = 5 if case["moments"] else 3 * (case["steps"] // case["obs_every"])
        return {"bytes": 2 * sites * per_site + 8 * rec * len(sizes),
                "flops": 2 * case["steps"] * sites * OPS_PER_UPDATE}
    sites = float(case["L"]) ** 2
    if kind == "exact_samples":
        # at least one doubling schedule from T0: top and bottom chains to 8 T0
        return {"bytes": case["samples"] * (sites / 8 + 8),
                "flops": 2 * 2 * 15 * case["T0"] * case["samples"] * sites * OPS_PER_UPDATE}
    if kind == "trajectories":
        return {"bytes": case["chains"] * (2 * case["steps"] + 2) * sites / 8,
                "flops": 2 * case["steps"] * case["chains"] * sites * OPS_PER_UPDATE}
    if kind == "counts":
        # five or nine popcounts and as many masks for 32 sites of a transition
        return {"bytes": case["chains"] * (2 * case["steps"] + 1) * sites / 8 + 96,
                "flops": 2 * case["steps"] * case["chains"] * sites / 32 * (10 if case["paired"] else 18)}
    if kind == "replicas":
        # the uniforms once per site, the comparison for 64 chains (2 words)
        per_site = (4.0 / 64.0 + 0.25) * 40.0 + 2 * 8 * 3
        return {"bytes": 3 * 8 * sites + 64 * 24, "flops": 2 * case["steps"] * sites * per_site}
    per_site = 1.0 if case["layout"] == "int8" else 0.125
    if kind == "table":
        steps = case["every"] * case["measurements"]
        return {"bytes": 2 * sites * per_site + 16 * (case["lmax"] + 1) * case["measurements"],
                "flops": 2 * steps * sites * OPS_PER_UPDATE +
                case["measurements"] * 2 * (case["lmax"] + 1) * sites / 32 * 3}
    if kind == "sweep":
        n = case["chains"]
        return {"bytes": n * (2 * sites * per_site + 24 * (case["steps"] // case["obs_every"]) +
                              8 * (case["rmax"] + 1)),
                "flops": n * (2 * case["steps"] * sites * OPS_PER_UPDATE + (case["rmax"] + 1) * sites / 32 * 3)}
    rec = case["steps"] // case["obs_every"] if case["obs_every"] else 0
    return {"bytes": 2 * sites * per_site + 24 * rec, "flops": 2 * case["steps"] * sites * OPS_PER_UPDATE}


def exact(case, seed):
    """LL and its gradient in 64 bits; every other kind's outputs are integers."""
    if case["kind"] != "ascent":
        return None
    v = _ascent_stats(case, seed)
    J, q = float(np.float32(case["at_J"])), float(np.float32(case["at_q"]))
    ll, gJ, gq = [], [], []
    for idx in range(3 if case["paired"] else 6):
        if case["paired"]:
            n, d = int(v[idx]), int(2 * v[3 + idx] - v[idx])
        else:
            n, d = int(v[2 * idx + 1] + v[2 * idx]), int(v[2 * idx + 1] - v[2 * idx])
        a, c = 2 * (idx >> 1) - 2, 2 * (idx & 1) - 1
        h = J * a + q * c
        ll += [d * h, -n * (abs(h) + math.log1p(math.exp(-2.0 * abs(h))))]
        resid = math.fsum([float(d), -n * math.tanh(h)])
        gJ.append(resid * a)
        gq.append(resid * c)
    return {"ll": np.float64(math.fsum(ll)), "grad": np.array([math.fsum(gJ), math.fsum(gq)])}
