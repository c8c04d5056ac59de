"""The work this library is measured on, through its public entry points.

Five kinds of pass:

  cycle      REWL cycles (rewl_run_cycles: sweeps, merge, exchange) of a
             batch of instances that is already running.  Returned: every
             walker's energy, histogram and ln g after the pass.
  create     a new context: layout, random lattices, energies, warm-up of
             every walker into its window.  Returned: as for a cycle.
  join       ln g joined over the windows and normalised, of every instance.
  thermo     <E> and C_V over a list of temperatures.
  jackknife  error bars of the joined ln g from a finished instance's pieces.

The cycles keep the launch plan that a program has: the default one of a
new context, or the one a tuned program sets.  ln f_final of the running
cases lies far below what any run reaches while it is measured, so that no
instance finishes (a finished one makes no more attempts).
The states behind join, thermo and jackknife are set up through the
workspace offsets that the library names for inspection and fault tools: a
density of states of the model's shape, a different offset for every
window, small differences between walkers, a nearly flat histogram, then one
merge.
"""
import math

import numpy as np
import torch

from paper_1402_2328_amd import rewl, workloads

RUNNING_LNF_FINAL = 1e-18
# algorithmic work of one attempt in lane operations (see bench.py)
OPS_PER_ATTEMPT = 126


def _case(name, kind, **kw):
    c = dict(kind=kind, model="ising", L=8, q=2, h=4, m=1, instances=1, flips=1000, cycles=1,
             schedule="halving", precision="fp64", page=0, temperatures=0)
    c.update(kw)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest run: one Ising L=8 instance of 4 walkers, one cycle of
        # 1000 attempts, where launches and one walker's chain are all
        _case("ising8_cycle", "cycle"),
        # the same run as a convergence loop issues it, many cycles per call
        _case("ising8_x8_cycles", "cycle", instances=8, cycles=16),
        # Ising L=32, 16 windows x 8 walkers, eight instances: the time to
        # converge of a few instances
        _case("ising32_x8", "cycle", L=32, h=16, m=8, instances=8, flips=10000),
        # the accuracy configuration: 64 walkers per window, 1/t schedule,
        # two-float FP32 ln g
        _case("ising32_m64_1t_fp32c", "cycle", L=32, h=16, m=64, instances=2, flips=10000,
              schedule="1t", precision="fp32c"),
        # a full chip: 1024 instances of Ising L=32 in the plan that the
        # tuner picks for them
        _case("ising32_x1024", "cycle", L=32, h=16, m=8, instances=1024, flips=10000, page=16),
        # one q=10 Potts L=20 instance, 32 windows x 16 walkers
        _case("potts10_x1", "cycle", model="potts", L=20, q=10, h=32, m=16, flips=10000),
        # a full chip of q=10 Potts in two-float FP32
        _case("potts10_x128_fp32c", "cycle", model="potts", L=20, q=10, h=32, m=16, instances=128,
              flips=10000, precision="fp32c"),
        # the uneven mix of 64 Ising and Potts instances in one fused launch
        _case("mix64", "cycle", model="mix", instances=64, flips=10000, page=64),
        # the same mix set up from nothing
        _case("mix64_create", "create", model="mix", instances=64),
        # results of a run: the joined ln g of eight Ising L=32 instances,
        _case("ising32_x8_join", "join", L=32, h=16, m=8, instances=8),
        # the specific heat of a q=10 Potts instance on a fine grid,
        _case("potts10_thermo", "thermo", model="potts", L=20, q=10, h=32, m=16, temperatures=2000),
        # and error bars of the accuracy configuration
        _case("ising32_m64_jackknife", "jackknife", L=32, h=16, m=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["cycle"] * 6 + ["create", "join", "thermo", "jackknife"])
    model = rng.choice(["ising", "ising", "potts"])
    if rng.random() < 0.35:
        L = rng.choice([16, 20, 32]) if model == "potts" else rng.choice([8, 16, 24, 32, 48, 64])
    else:
        L = 2 * _log_int(rng, 3, 32 if model == "ising" else 16)
    q = rng.randint(2, 20) if model == "potts" else 2
    nbins = L * L + 1 if model == "ising" or q == 2 else 2 * L * L + 1
    h = min(_log_int(rng, 1, 48), max(1, nbins // 12))
    m = _log_int(rng, 1, 64)
    c = dict(model=model, L=L, q=q, h=h, m=m, precision=rng.choice(["fp64", "fp64", "fp32c"]),
             schedule=rng.choice(["halving", "halving", "1t"]))
    if h == 1 and rng.random() < 0.5:
        c["L"] = L + 1 if L < 32 else L - 1        # one window takes odd lattices as well
    if kind == "cycle":
        walkers = _log_int(rng, max(h * m, 4), max(h * m, 65536))
        # at most 1.2 GB of state (20 bytes per bin, the spins)
        per = h * m * (20 * (nbins / (1 + (h - 1) / 4) + 2) + L * L)
        inst = max(1, min(walkers // (h * m), int(1.2e9 / per), 2048))
        attempts = 3e8 / (h * m * inst)
        flips = max(200, min(_log_int(rng, 500, 10000), int(attempts)))
        cycles = 4 if flips <= 2500 and rng.random() < 0.5 else 1
        return _case("", "cycle", instances=inst, flips=flips, cycles=cycles, **c)
    c["schedule"] = "halving"
    if kind == "create":
        inst = max(1, min(_log_int(rng, 1, 64), 8192 // (h * m)))
        return _case("", "create", instances=inst, **c)
    if kind == "join":
        return _case("", "join", instances=_log_int(rng, 1, 16), **c)
    if kind == "thermo":
        return _case("", "thermo", temperatures=_log_int(rng, 20, 2000), **c)
    return _case("", "jackknife", **dict(c, m=max(2, m)))


# ---- parameters ----

def _configs(case, seed, lnf_final=RUNNING_LNF_FINAL):
    if case["model"] == "mix":
        cfgs = workloads.batched_mix(case["instances"])
        for c in cfgs:
            c["seed"] += 1000 * seed
    else:
        one = workloads.config(
            workloads.ISING if case["model"] == "ising" else workloads.POTTS, case["L"], q=case["q"],
            n_windows=case["h"], walkers_per_window=case["m"], flips=case["flips"], seed=seed + 1,
            precision=workloads.FP64 if case["precision"] == "fp64" else workloads.FP32C,
            schedule=workloads.HALVING if case["schedule"] == "halving" else workloads.ONE_OVER_T)
        cfgs = workloads.replicated(one, case["instances"])
    return [dict(c, lnf_final=lnf_final) for c in cfgs]


def _views(ctx):
    """Energies, histograms and ln g (FP32C: its high parts) of all walkers,
    as views of the workspace at the offsets the library names."""
    n = len(ctx.params)
    last = ctx.geometry[-1]["h"] * ctx.geometry[-1]["m"] - 1
    a, b = ctx.locate_walker(0, 0), ctx.locate_walker(n - 1, last)
    walkers = sum(g["h"] * g["m"] for g in ctx.geometry)
    bins = sum(int((g["hi"] - g["lo"] + 1).sum()) * g["m"] for g in ctx.geometry)
    lng = torch.float64 if ctx.params[0].precision == rewl.FP64 else torch.float32
    size = 8 if lng == torch.float64 else 4
    for key, count, width, tail in (("energy", walkers, 4, 1), ("H", bins, 4, b["n_bins"]),
                                    ("lng", bins, size, b["n_bins"])):
        if b[key] - a[key] != width * (count - tail):
            raise RuntimeError(f"{key} of the walkers is not one array")
    ws = ctx.workspace
    return {"energy": ws[a["energy"]:a["energy"] + 4 * walkers].view(torch.int32),
            "H": ws[a["H"]:a["H"] + 4 * bins].view(torch.int32),
            "lng": ws[a["lng"]:a["lng"] + size * bins].view(lng)}


# ---- synthetic results of a run (join, thermo, jackknife) ----

def _true_lng(model, N, q, nbins):
    """A density of states of the model's shape."""
    x = np.linspace(0.0, 1.0, nbins)
    s, t = np.clip(1.0 - x, 1e-300, 1.0), np.clip(x, 1e-300, 1.0)   # satisfied, broken bonds
    if model == "ising" or q == 2:
        return N * (-s * np.log(s) - t * np.log(t))
    p = 1.0 / q
    return N * (math.log(q) - s * np.log(s / p) - t * np.log(t / (1.0 - p)))


def _visited(model, q, nbins):
    """Every bin but those that no even lattice reaches, just above the ground
    state (and, symmetric, below the top)."""
    U = np.ones(nbins, bool)
    if model == "ising" or q == 2:
        U[1] = U[-2] = False
    else:
        U[1:4] = False
    return U


def _windows(nbins, h):
    """The equal-size split with 75 % overlap."""
    S, D = nbins - 1, 4 + (h - 1)
    return ([(2 * i * S + D) // (2 * D) for i in range(h)],
            [(2 * (i + 4) * S + D) // (2 * D) for i in range(h)])


def _geometry(case):
    N = case["L"] ** 2
    two = case["model"] == "ising" or case["q"] == 2
    nbins = (N if two else 2 * N) + 1
    binw = 4 if case["model"] == "ising" else (2 if two else 1)
    return N, nbins, binw


def _rows(case, seed):
    """Per instance and window the walkers' ln g [m, bins] and H."""
    rng = np.random.default_rng(seed)
    N, nbins, _ = _geometry(case)
    lng = _true_lng(case["model"], N, case["q"], nbins)
    U = _visited(case["model"], case["q"], nbins)
    lo, hi = _windows(nbins, case["h"])
    out = []
    for _ in range(case["instances"]):
        rows = []
        for w in range(case["h"]):
            seen = U[lo[w]:hi[w] + 1]
            l = lng[lo[w]:hi[w] + 1] - lng[lo[w]] + 1000.0 + 100.0 * rng.random()
            l = l - min(0.0, float(l.min())) + 0.01 * rng.standard_normal((case["m"], l.size))
            h = rng.integers(2000, 2100, l.shape)
            l, h = np.where(seen, l, 0.0), np.where(seen, h, 0)
            if case["precision"] == "fp32c":
                l = l.astype(np.float32).astype(np.float64)
            rows.append((l, h.astype(np.int32)))
        out.append(rows)
    return out


def _temperatures(case):
    lo, hi = (1.0, 4.0) if case["model"] == "ising" else (0.4, 1.6)
    return np.linspace(lo, hi, case["temperatures"])


# ---- the passes ----

def prepare(case, seed):
    kind = case["kind"]
    state = {"kind": kind, "case": case}
    if kind == "create":
        state["params"] = [workloads.rewl_params_of(c) for c in _configs(case, seed)]
        return state
    lnf_final = 0.6 if kind == "jackknife" else RUNNING_LNF_FINAL
    ctx = rewl.Context([workloads.rewl_params_of(c) for c in _configs(case, seed, lnf_final)])
    state.update(ctx=ctx, out=_views(ctx))
    if kind == "cycle":
        if case["page"]:
            fused = case["model"] == "mix"
            ctx.set_launch(page_bins=case["page"], rng_producer=0, potts_nibbles=2 if fused else -1)
            if fused:
                ctx.set_batching(fused=1)
        ctx.run_cycles(1, min(case["flips"], 2000))
        return state
    rows = _rows(case, seed)
    lng = np.concatenate([l.reshape(-1) for inst in rows for l, _ in inst])
    H = np.concatenate([h.reshape(-1) for inst in rows for _, h in inst])
    state["out"]["lng"].copy_(torch.from_numpy(lng))
    state["out"]["H"].copy_(torch.from_numpy(H))
    ctx.merge()
    if kind == "thermo":
        state["T"] = _temperatures(case)
    return state


def run(state):
    kind, case = state["kind"], state["case"]
    if kind == "cycle":
        state["ctx"].run_cycles(case["cycles"], case["flips"], use_graph=case["cycles"] > 1)
        return state["out"]
    if kind == "create":
        ctx = rewl.Context(state["params"])
        state["ctx"] = ctx
        return _views(ctx)
    ctx = state["ctx"]
    if kind == "join":
        return [dict(zip(("lng", "joins"), ctx.get_lng(i))) for i in range(case["instances"])]
    if kind == "thermo":
        return dict(zip(("E", "Cv"), ctx.thermo(state["T"])))
    return dict(zip(("mean", "err"), ctx.jackknife(0)))


def work(case):
    if case["model"] == "mix":
        cfgs = workloads.batched_mix(case["instances"])
        shapes = [("ising" if c["model"] == workloads.ISING else "potts", c["L"], c["q"], c["n_windows"],
                   c["walkers_per_window"]) for c in cfgs]
    else:
        shapes = [(case["model"], case["L"], case["q"], case["h"], case["m"])] * case["instances"]
    walkers = spins = bins = 0
    for model, L, q, h, m in shapes:
        two = model == "ising" or q == 2
        lo, hi = _windows((L * L if two else 2 * L * L) + 1, h)
        walkers += h * m
        spins += h * m * L * L
        bins += m * sum(b - a + 1 for a, b in zip(lo, hi))
    if case["kind"] == "cycle":
        # spins, ln g and H read and written once
        return {"bytes": 2 * case["cycles"] * (spins + 12 * bins),
                "flops": case["cycles"] * case["flips"] * walkers * OPS_PER_ATTEMPT}
    if case["kind"] == "create":
        # spins, ln g and H written once; each spin drawn and its two bonds counted
        return {"bytes": spins + 12 * bins, "flops": 20 * spins}
    nbins = _geometry(case)[1]
    if case["kind"] == "join":
        return {"bytes": 8 * (bins + case["instances"] * nbins), "flops": bins}
    if case["kind"] == "thermo":
        # two weights of about 20 operations per bin and temperature
        return {"bytes": 8 * (bins + nbins + 3 * case["temperatures"]),
                "flops": 40 * nbins * case["temperatures"] + bins}
    # one mean over the others per walker and bin from shared sums
    return {"bytes": 8 * (bins + 2 * nbins), "flops": 2 * bins + 10 * case["m"] * nbins}


# ---- the same results from plain numpy in 64 bits ----

def _pairwise_mean(v):
    """Mean over rows, summed pairwise in row order."""
    n = len(v)
    v = list(v)
    while len(v) > 1:
        v = [v[i] + v[i + 1] if i + 1 < len(v) else v[i] for i in range(0, len(v), 2)]
    return v[0] / n


def _join(case, reps):
    """Joins the windows' representatives where their five-point slopes agree
    best and normalises."""
    N, nbins, _ = _geometry(case)
    U = _visited(case["model"], case["q"], nbins)
    lo, hi = _windows(nbins, case["h"])
    R = np.full(nbins, -np.inf)
    R[lo[0]:hi[0] + 1] = reps[0]
    shift, joins = 0.0, []

    def slope(l, at, b):
        j = b - at
        return (((l[j - 2] - 8.0 * l[j - 1]) + 8.0 * l[j + 1]) - l[j + 2]) / 12.0

    for w in range(1, case["h"]):
        la, lb = reps[w - 1], reps[w]
        b = np.arange(lo[w] + 2, hi[w - 1] - 1)
        b = b[np.all([U[b + d] for d in range(-2, 3)], axis=0)] if b.size else b
        if b.size:
            at = int(b[np.argmin(np.abs(slope(la, lo[w - 1], b) - slope(lb, lo[w], b)))])
        else:
            at = (lo[w] + hi[w - 1]) // 2
        shift = (la[at - lo[w - 1]] + shift) - lb[at - lo[w]]
        R[at:hi[w] + 1] = lb[at - lo[w]:] + shift
        joins.append(at)
    R[~U] = -np.inf
    if case["model"] == "ising":
        mx = R.max()
        R = R + (N * math.log(2.0) - (mx + math.log(np.exp(R - mx).sum())))
    else:
        R = R + (math.log(case["q"]) - R[0])
    return R, np.array(joins, np.int32)


def exact(case, seed):
    if case["kind"] in ("cycle", "create"):
        return None     # a stochastic trajectory: whole numbers, compared as such
    rows = _rows(case, seed)
    if case["kind"] == "jackknife":
        m = case["m"]
        keep = [[i for i in range(m) if i != k] for k in range(m)]
        R = np.array([_join(case, [_pairwise_mean(l[keep[k]]) for l, _ in rows[0]])[0] for k in range(m)])
        fin = np.isfinite(R).all(axis=0)
        mean, err = np.full(R.shape[1], -np.inf), np.zeros(R.shape[1])
        mean[fin] = R[:, fin].mean(axis=0)
        err[fin] = np.sqrt((m - 1) / m * ((R[:, fin] - mean[fin]) ** 2).sum(axis=0))
        return {"mean": mean, "err": err}
    joined = [_join(case, [_pairwise_mean(l) for l, _ in inst]) for inst in rows]
    if case["kind"] == "join":
        return [{"lng": R, "joins": None} for R, _ in joined]
    N, nbins, binw = _geometry(case)
    E = -2.0 * N + binw * np.arange(nbins)
    T = _temperatures(case)
    Em, Cv = np.zeros(len(T)), np.zeros(len(T))
    for i, t in enumerate(T):
        a = joined[0][0] - E / t
        wgt = np.exp(a - a.max())
        Em[i] = (wgt * E).sum() / wgt.sum()
        Cv[i] = (wgt * (E - Em[i]) ** 2).sum() / wgt.sum() / t ** 2
    return {"E": Em, "Cv": Cv}
