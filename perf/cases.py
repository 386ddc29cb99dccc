"""Workloads whose speed is tracked: the calibration replay through its public entry points.

Four paths, each over the range a calibration service uses:

``grid``        kvr_cost_grid on one wait sample, BRUTE or SORTED (CostGridCall: the buffers
                are kept and each pass only enqueues work, as a serving loop does), optionally
                followed by kvr_select_policy
``boot``        the bootstrap over resamples, brute force or factored (BootstrapCall)
``replay``      kvr_capacity_replay of request sequences under several host timers
``controller``  kvr_controller_select (ControllerCall)

Inputs are drawn on the GPU from the seed with the laws of ``workloads.py`` (the approval-wait
families and context sizes); prices come from its platform constants.
"""
import math

import numpy as np
import torch

import paper_2608_30830_amd as kvr

HBM, LINK, PREFILL, C2, WREF = 250e9, 50e9, 20000.0, 425.0, 1800.0
LAM_CRIT = C2 / WREF
KV = {"mix": 131072.0, "exp": 131072.0, "weibull": 327680.0}
REPLAY_PRICES = (0.0176, 0.02, 1.91)      # alpha_1, beta_2, beta_3 of one request (H100 NVL)
FAMILIES = ("lognormal", "exponential", "mixture")


def listed():
    return [
        # one agent's calibration sample: the smallest call, latency only
        dict(name="grid-tiny-brute", kind="grid", law="exp", n=1000, k1=1, k2=65, loads=4,
             method="brute", perm=False, select=False, charge=False),
        # an ordinary calibration sample with the whole selection
        dict(name="grid-64k-brute-select", kind="grid", law="mix", n=65536, k1=1, k2=257, loads=16,
             method="brute", perm=False, select=True, charge=False),
        # a fleet's sample by brute force: a million waits, 64 loads
        dict(name="grid-1m-brute", kind="grid", law="weibull", n=1 << 20, k1=1, k2=1025, loads=64,
             method="brute", perm=False, select=False, charge=False),
        # an ordinary odd-sized sample by the sorted closed form, two-tier timers, the copy at
        # offload charged
        dict(name="grid-100k-sorted", kind="grid", law="mix", n=100003, k1=5, k2=101, loads=7,
             method="sorted", perm=False, select=True, charge=True),
        # a fleet's sample with the order of its waits wanted too
        dict(name="grid-1m-sorted-order", kind="grid", law="weibull", n=1 << 20, k1=1, k2=1025,
             loads=64, method="sorted", perm=True, select=False, charge=False),
        # the largest sample
        dict(name="grid-16m-sorted", kind="grid", law="weibull", n=1 << 24, k1=1, k2=65, loads=4,
             method="sorted", perm=False, select=False, charge=False),
        # few resamples of a small odd-sized sample, the whole cost tensor wanted
        dict(name="boot-37x5003-cost", kind="boot", law="mix", n=5003, rows=37, m=5003, k1=9, k2=41,
             loads=7, factored=False, cost=True),
        # the one-tier bootstrap by brute force
        dict(name="boot-1024x64k", kind="boot", law="mix", n=65536, rows=1024, m=65536, k1=1, k2=257,
             loads=16, factored=False, cost=False),
        # the two-tier bootstrap by brute force, the benchmark's step at an eighth of its rows
        dict(name="boot-twotier-512x64k", kind="boot", law="mix", n=65536, rows=512, m=65536, k1=64,
             k2=257, loads=32, factored=False, cost=False),
        # the two-tier bootstrap at its full size by the factored closed form
        dict(name="boot-twotier-factored", kind="boot", law="mix", n=65536, rows=4096, m=65536, k1=64,
             k2=257, loads=32, factored=True, cost=False),
        # the finite-capacity replay behind Table 6 as a batch that fills the GPU
        dict(name="replay-8192x4000", kind="replay", family="exponential", rate=2.0, reps=8192,
             n=4000, timers=5, ctx=False),
        # the controller on a hundred calibration sequences, contexts of different sizes
        dict(name="controller-100x4000", kind="controller", family="mixture", rate=2.0, reps=100,
             n=4000, ctx=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("grid-brute", "grid-sorted", "boot", "boot-factored", "replay", "controller"))
    law = rng.choice(("mix", "exp", "weibull"))
    if kind == "grid-brute":
        n, k1, k2, loads = _log(rng, 300, 1 << 20), rng.choice((1, 1, 1, 4, 13)), _log(rng, 16, 1025), _log(rng, 2, 64)
        return dict(kind="grid", law=law, n=n, k1=k1, k2=k2, loads=loads, method="brute", perm=False,
                    select=rng.random() < 0.5, charge=rng.random() < 0.3)
    if kind == "grid-sorted":
        n, k1, k2, loads = _log(rng, 1500, 1 << 24), rng.choice((1, 1, 3, 16)), _log(rng, 16, 1025), _log(rng, 2, 64)
        return dict(kind="grid", law=law, n=n, k1=k1, k2=k2, loads=loads, method="sorted",
                    perm=rng.random() < 0.3, select=rng.random() < 0.5, charge=rng.random() < 0.3)
    if kind in ("boot", "boot-factored"):
        n, rows = _log(rng, 1000, 65536), _log(rng, 16, 1024)
        m = n if rng.random() < 0.7 else max(500, n // 2 + 1)
        k1, k2, loads = _log(rng, 1, 64), _log(rng, 24, 257), _log(rng, 3, 32)
        rows = max(1, min(rows, 512 * 65536 * 64 * 257 * 32 // (m * k1 * k2 * loads)))
        return dict(kind="boot", law=law, n=n, rows=rows, m=m, k1=k1, k2=k2, loads=loads,
                    factored=kind == "boot-factored",
                    cost=rows * loads * k1 * k2 < (1 << 24) and rng.random() < 0.4)
    family, rate = rng.choice(FAMILIES), rng.choice((0.5, 1.0, 2.0, 3.0))
    if kind == "replay":
        reps, n = _log(rng, 1, 4096), _log(rng, 200, 8192)
        return dict(kind="replay", family=family, rate=rate, reps=reps, n=n, timers=rng.randint(1, 8),
                    ctx=rng.random() < 0.5)
    reps, n = _log(rng, 3, 8192), _log(rng, 200, 8192)
    return dict(kind="controller", family=family, rate=rate, reps=max(1, min(reps, (1 << 25) // n)),
                n=n, ctx=rng.random() < 0.5)


# ---- inputs -------------------------------------------------------------------------------

def _rand(gen, *shape):
    return torch.rand(*shape, generator=gen, dtype=torch.float64, device="cuda")


def _randn(gen, *shape):
    return torch.randn(*shape, generator=gen, dtype=torch.float64, device="cuda")


def _expo(gen, mean, *shape):
    return -mean * torch.log1p(-_rand(gen, *shape))


def _sample(law, n, gen):
    """Waits (s) and context sizes (tokens) of one calibration sample."""
    if law == "mix":
        short = _rand(gen, n) < 0.7
        z = _randn(gen, n)
        w = torch.where(short, 60.0 * torch.exp(z), 7200.0 * torch.exp(0.8 * z))
        t = torch.randint(2048, 32769, (n,), generator=gen, dtype=torch.int32, device="cuda")
    elif law == "exp":
        w = _expo(gen, 1800.0, n)
        t = torch.full((n,), 8192, dtype=torch.int32, device="cuda")
    else:
        cap = -math.expm1(-(86400.0 / 1800.0) ** 0.5)
        w = 1800.0 * torch.log1p(-_rand(gen, n) * cap) ** 2
        t = torch.clamp(torch.round(16384.0 * torch.exp(0.7 * _randn(gen, n))), 1024, 131072).to(torch.int32)
    return w, t


def _family(family, gen, *shape):
    """The approval-wait families of the finite-capacity replay, mean 1,800 s each."""
    if family == "lognormal":
        return torch.exp(math.log(1800.0) - 0.5 + _randn(gen, *shape))
    if family == "exponential":
        return _expo(gen, 1800.0, *shape)
    short = _rand(gen, *shape) < 0.5
    return torch.where(short, _expo(gen, 60.0, *shape),
                       torch.exp(math.log(3540.0) - 0.245 + 0.7 * _randn(gen, *shape)))


def _timers(case):
    k1, k2, loads = case["k1"], case["k2"], case["loads"]
    t1 = [0.0] if k1 == 1 else [float(x) for x in np.geomspace(1.0, 3600.0, k1)]
    t2 = [float(x) for x in np.geomspace(10.0, 86400.0, k2 - 1)] + [math.inf]
    lam = [float(x) for x in np.linspace(0.05, 1.0, loads)] if loads > 1 else [2.0 * LAM_CRIT]
    return t1, t2, lam


def _prices(case):
    return kvr.kvr_prices_from_platform(KV[case["law"]], HBM, LINK, PREFILL, 1.0, C2, WREF,
                                        charge_offload=bool(case.get("charge")))


def _replay_prices():
    p = kvr.kvr_prices()
    p.a1_per_token, p.b2_per_token, p.b3_per_token = REPLAY_PRICES
    p.host_slots_c2, p.w_ref_s, p.offload_per_token = C2, WREF, 0.0
    return p


def _eq3(rate):
    """The load-indexed host timer at rate x the critical load (inf at or below it)."""
    _, b2, b3 = REPLAY_PRICES
    a2 = max(0.0, rate * LAM_CRIT - LAM_CRIT) * b3 / C2
    return (b3 - b2) / a2 if a2 > 0.0 else math.inf


def _replay_timers(case):
    """Table 6's columns: fixed timers, the load-indexed one, host-retain."""
    return ([600.0, 1800.0, 5400.0, _eq3(case["rate"]), math.inf, 120.0, 300.0, 14400.0])[:case["timers"]]


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind = case["kind"]
    if kind in ("grid", "boot"):
        w, t = _sample(case["law"], case["n"], gen)
        grid = kvr.PolicyGrid(*_timers(case))
        if kind == "grid":
            method = kvr.KVR_BRUTE if case["method"] == "brute" else kvr.KVR_SORTED
            call = kvr.CostGridCall(w, t, _prices(case), grid, method, want_perm=case["perm"])
        else:
            idx = torch.randint(0, case["n"], (case["rows"], case["m"]), generator=gen,
                                dtype=torch.int32, device="cuda")
            call = kvr.BootstrapCall(w, t, idx, _prices(case), grid, want_cost=case["cost"],
                                     factored=case["factored"])
        return {"case": case, "call": call, "grid": grid}
    shape = (case["reps"], case["n"])
    arrival = torch.cumsum(_expo(gen, 1.0 / (case["rate"] * LAM_CRIT), *shape), dim=1)
    # a parallel cumsum may round a later instant below an earlier one
    arrival = torch.cummax(arrival, dim=1).values.contiguous()
    wait = _family(case["family"], gen, *shape)
    ctx = torch.randint(2048, 32769, shape, generator=gen, dtype=torch.int32,
                        device="cuda") if case["ctx"] else None
    state = {"case": case, "arrival": arrival, "wait": wait, "ctx": ctx, "prices": _replay_prices()}
    if kind == "controller":
        state["call"] = kvr.ControllerCall(arrival, wait, state["prices"], case["rate"] * LAM_CRIT, ctx)
    else:
        state["timers"] = _replay_timers(case)
    return state


# ---- one pass -----------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "replay":
        cost, restored, admitted = kvr.kvr_capacity_replay(
            state["arrival"], state["wait"], state["prices"], state["timers"], state["ctx"],
            check=False)
        return {"cost": cost, "restored": restored, "admitted": admitted}
    call = state["call"]
    call.launch()
    if kind == "controller":   # eight 64-bit integers, then seven doubles
        return {"whole": call.out[:64].view(torch.int64), "real": call.out[64:].view(torch.float64)}
    if kind == "grid":
        out = {"cost": call.cost}
        if case["perm"]:
            out["order"] = call.perm
        if case["select"]:
            out["best"], out["best_cost"], out["branch"] = kvr.kvr_select_policy(
                call.cost, bool(state["grid"].last_inf))
        return out
    out = {"best": call.best, "best_cost": call.best_cost}
    if case["cost"]:
        out["cost"] = call.cost
    return out


def work(case):
    """Inputs once, outputs once.  Brute force is asked for every evaluation (one multiply-add
    each); the closed forms and the replay need about the operations below."""
    kind, n = case["kind"], case["n"]
    if kind in ("grid", "boot"):
        P, L = case["k1"] * case["k2"], case["loads"]
        if kind == "grid":
            nbytes = 12 * n + 8 * P * L + (4 * n if case["perm"] else 0)
            flops = 2 * n * P * L if case["method"] == "brute" else 2 * n + 8 * P * L
        else:
            rows, m = case["rows"], case["m"]
            nbytes = 12 * n + 4 * rows * m + 12 * rows * L + (8 * rows * L * P if case["cost"] else 0)
            flops = 2 * rows * (2 * m + 4 * P * L) if case["factored"] else 2 * rows * m * P * L
        return {"bytes": nbytes, "flops": flops}
    reps, timers = case["reps"], case["timers"] if kind == "replay" else 2
    nbytes = reps * n * (20 if case["ctx"] else 16) + (24 * reps * timers if kind == "replay" else 120)
    return {"bytes": nbytes, "flops": reps * n * (1 + timers)}


def tolerance(case):
    # binary64 sums of up to 2^24 positive terms in another order; a selection may differ only
    # where two policies' costs agree to rounding.  The replay counts whole tokens and requests
    # and forms each cost from them in a few roundings.
    if case["kind"] in ("replay", "controller"):
        return {"rel": 1e-15, "max": 1e-14, "differ": 0.0}
    # Measured against exact(): rel up to 2.2e-15 (65,536 terms added one after another).
    return {"rel": 1e-14, "max": 1e-13, "differ": 1e-3}


# ---- the same results in plain torch --------------------------------------------------------

def _costs(case, N, S, query, t1, e, dev):
    """m * C for [rows, L, P] from prefix sums N, S ([rows, positions + 1])."""
    u1, ue = query
    p = {"a1": KV[case["law"]] / HBM, "b2": KV[case["law"]] / LINK, "b3": 1.0 / PREFILL}
    off = p["b2"] if case.get("charge") else 0.0
    k1, k2 = len(t1), e.shape[1]
    N1, S1 = N[:, u1].repeat_interleave(k2, 1), S[:, u1].repeat_interleave(k2, 1)
    Ne, Se, Nt = N[:, ue], S[:, ue], N[:, -1:]
    tt = torch.tensor(t1, dtype=torch.float64, device=dev).repeat_interleave(k2)
    ee = e.reshape(-1)
    held = torch.where(torch.isinf(ee), torch.zeros_like(ee), ee - tt)
    fixed = p["a1"] * (S1 + tt * (Nt - N1)) + (p["b2"] + off) * (Ne - N1) + (p["b3"] + off) * (Nt - Ne)
    hold = (Se - S1) - tt * (Ne - N1) + held * (Nt - Ne)
    lam = _timers(case)[2]
    a2 = torch.tensor([max(0.0, x - LAM_CRIT) * p["b3"] / C2 for x in lam], dtype=torch.float64, device=dev)
    return fixed[:, None, :] + a2[None, :, None] * hold[:, None, :]


def _exact_grid(case, seed):
    state = prepare(case, seed)
    call = state["call"]
    w, order = torch.sort(call.wait_s)
    T = call.ctx.double()[order]
    dev = w.device
    t1, t2, lam = _timers(case)
    t1v = torch.tensor(t1, dtype=torch.float64, device=dev)
    e = t1v[:, None] + torch.tensor(t2, dtype=torch.float64, device=dev)[None, :]
    u1 = torch.searchsorted(w, t1v, right=True)
    ue = torch.searchsorted(w, e.reshape(-1), right=True)
    k1, k2, L = len(t1), len(t2), len(lam)

    def prefix(x):
        return torch.cat([torch.zeros(x.shape[0], 1, dtype=torch.float64, device=dev),
                          torch.cumsum(x, dim=1)], dim=1)

    if case["kind"] == "grid":
        N, S = prefix(T[None]), prefix((T * w)[None])
        cost = (_costs(case, N, S, (u1, ue), t1, e, dev)[0] / case["n"]).reshape(L, k1, k2)
        out = {"cost": cost}
        if case["perm"]:
            out["order"] = None
        if case["select"]:
            out["best"], out["branch"] = None, None
            out["best_cost"] = cost.reshape(L, -1).min(dim=1).values
        return out
    rank = torch.empty_like(order)
    rank[order] = torch.arange(len(order), device=dev)
    rows, m, n = case["rows"], case["m"], case["n"]
    step = max(1, min(rows, int(2 ** 26 // max(n, k1 * k2 * L))))
    best_cost, costs = [], []
    for r0 in range(0, rows, step):
        idx = rank[call.idx[r0:r0 + step].long()]
        at = idx + n * torch.arange(idx.shape[0], device=dev)[:, None]
        c = torch.bincount(at.reshape(-1), minlength=idx.shape[0] * n).reshape(-1, n).double()
        cost = _costs(case, prefix(c * T), prefix(c * T * w), (u1, ue), t1, e, dev) / m
        best_cost.append(cost.min(dim=2).values)
        if case["cost"]:
            costs.append(cost.reshape(-1, L, k1, k2))
    out = {"best": None, "best_cost": torch.cat(best_cost)}
    if case["cost"]:
        out["cost"] = torch.cat(costs)
    return out


def _replay_counts(state, timers):
    """(restored tokens, admissions), each [reps, timers], one request of every sequence at a time."""
    a, w, ctx = state["arrival"], state["wait"], state["ctx"]
    reps, n = a.shape
    T = torch.ones_like(w, dtype=torch.int64) if ctx is None else ctx.long()
    later = torch.arange(1, n + 1, device=a.device)
    restored, admitted = [], []
    for t2 in timers:
        stays = w <= t2
        leave = torch.where(stays, a + w, a + t2)
        freed_at = torch.maximum(torch.searchsorted(a, leave.contiguous()), later).t().contiguous()
        freed = torch.zeros(n + 1, reps, dtype=torch.int64, device=a.device)
        got = torch.empty(n, reps, dtype=torch.bool, device=a.device)
        occ = torch.zeros(reps, dtype=torch.int64, device=a.device)
        for j in range(n):
            occ = occ - freed[j]
            fits = occ < int(C2)
            occ = occ + fits
            freed.scatter_add_(0, freed_at[j][None], fits.long()[None])
            got[j] = fits
        got = got.t()
        restored.append((T * (got & stays)).sum(dim=1))
        admitted.append(got.sum(dim=1))
    return torch.stack(restored, 1), torch.stack(admitted, 1), T


def exact(case, seed):
    if case["kind"] in ("grid", "boot"):
        return _exact_grid(case, seed)
    state = prepare(case, seed)
    a1, b2, b3 = REPLAY_PRICES
    n = case["n"]
    if case["kind"] == "replay":
        restored, admitted, T = _replay_counts(state, state["timers"])
        total = T.sum(dim=1, keepdim=True)
        cost = (b2 * restored.double() + b3 * (total - restored).double()) / n
        return {"cost": cost, "restored": restored, "admitted": admitted}
    timers = (_eq3(case["rate"]), math.inf)
    restored, admitted, T = _replay_counts(state, timers)
    R, total = restored.sum(dim=0).double(), T.sum().double()
    cost = b2 * R + b3 * (total - R)
    N = case["reps"] * n
    t_star = b3 / a1
    short = (state["wait"] <= t_star).sum().double()
    dev = R.device
    real = torch.cat([torch.tensor([timers[0]], dtype=torch.float64, device=dev), cost, cost / N,
                      torch.tensor([t_star], dtype=torch.float64, device=dev), (short / N)[None]])
    return {"whole": None, "real": real}
