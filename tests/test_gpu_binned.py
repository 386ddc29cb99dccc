"""GPU parity of KVR_SORTED without a requested order (per-bin sums over the
grid's thresholds) where it can go wrong: numbers of thresholds around every
power of two that sizes the search and at the bin ranges, samples around the
block and chunk sizes, waits on thresholds, equal and infinite thresholds,
one crowded bin, the largest context sizes, and grids beyond the path's limit.

Tolerance: the per-bin sums are exact up to 2^-64 of a bin's width per wait, and four
roundings bring one to binary64.  A prefix sum passes it through at most 4 additions in a
thread (4,096 bins), 6 in the wave's tree and 16 of wave totals, or, in tiles of 1,024
bins, 1 + 6 + 16 and 33 of tile totals (32,980 bins at most): 60 roundings, 80 with the
closed form's own, all of sums of terms of one sign.  So every cost is within 80 * 2^-53
of the sum of its terms' magnitudes:
(a1 t1 + a2 min(e, max w) + b2 + b3) * tokens / n (the last three only for
timers that some wait passes), doubled for the terms that are
differences of two prefix sums."""
import numpy as np
import pytest

import workloads
from tests import helpers as H
from tests.test_gpu_parity import _dev, _f64, _i32, _lib_prices, _np, assert_selection

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kvr():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2608_30830_amd as k
    k.load_library()
    return k


def _bound(pr, wl):
    a2 = np.maximum(0.0, wl.lam - pr.c2 / pr.w_ref) * pr.b3 / pr.c2
    wmax = wl.wait_s.max()
    with np.errstate(over="ignore"):     # deadlines may overflow to infinity
        e = np.minimum(wl.t1[:, None] + wl.t2[None, :], wmax)
    t1 = np.minimum(wl.t1, wmax)
    # past the longest wait no request pays a host term: exact zeros, not differences
    host = (a2[:, None, None] * (e + t1[:, None])[None] + pr.b2 + pr.b3) * (wl.t1 < wmax)[None, :, None]
    per = pr.a1 * t1[None, :, None] + host
    # a few roundings to multiples of the smallest denormal, where the costs are that small
    return (2.0 * 80.0 * H.EPS * per * float(wl.ctx_tokens.astype(np.float64).sum()) / wl.n
            + 4 * 5e-324)


def _check(kvr, oracle_mod, wl):
    pr = oracle_mod.workload_prices(wl)
    g = kvr.PolicyGrid(wl.t1, wl.t2, wl.lam)
    w, T = _dev(wl.wait_s, _f64()), _dev(wl.ctx_tokens, _i32())
    cost = kvr.kvr_cost_grid(w, T, _lib_prices(kvr, wl), g, method=kvr.KVR_SORTED)
    again = kvr.kvr_cost_grid(w, T, _lib_prices(kvr, wl), g, method=kvr.KVR_SORTED)
    same = np.array_equal(_np(cost), _np(again))        # no order of atomics can show
    assert same
    ref = oracle_mod.cost_grid(wl.wait_s, wl.ctx_tokens, pr, wl.t1, wl.t2, wl.lam)
    worst = float((np.abs(_np(cost) - ref) / _bound(pr, wl)).max())
    assert worst <= 1.0, f"{worst:.3g} times the bound"
    best, _, _ = kvr.kvr_select_policy(cost, g.last_inf)
    assert_selection(ref, _np(best), oracle_mod.select(ref, wl.t2)[0])
    return _np(cost)


# bins = K1 + K1*K2 + 211 fixed edges + 1 around 512 and 2,048 (search sizes),
# 4,095 (one range) and 4,096 (fused prefix), two and more ranges; K1 > K2; K2 = 1
@pytest.mark.parametrize("k1,k2", [(1, 1), (1, 298), (1, 299), (1, 300), (1, 1834), (1, 1835),
                                   (1, 1836), (1, 3881), (1, 3882), (1, 3883), (1, 3884),
                                   (8, 1023), (64, 130), (130, 64), (300, 1), (16, 1024),
                                   (16384, 1)])
def test_threshold_counts(kvr, oracle_mod, k1, k2):
    _check(kvr, oracle_mod, workloads.random_case(700 + k1 + k2, 2500, k1, k2, 3, ties=True,
                                                     inf_last=k2 > 1))


# one block sorts up to 2,048 waits, the cheaper way beyond 48 rows and columns of deadlines
@pytest.mark.parametrize("n,k1,k2", [(1, 49, 49), (2048, 49, 49), (2049, 49, 49), (2048, 48, 51),
                                     (2048, 51, 48), (1000, 49, 330), (1000, 330, 49)])
def test_small_samples_of_many_rows(kvr, oracle_mod, n, k1, k2):
    _check(kvr, oracle_mod, workloads.random_case(53 + n, n, k1, k2, 3, ties=n > 4))


@pytest.mark.parametrize("n", [1, 2, 1023, 1024, 1025, 4097, 262144, 262145, 1048577])
def test_sample_sizes(kvr, oracle_mod, n):
    _check(kvr, oracle_mod, workloads.random_case(41, n, 2, 9, 2, ties=n > 4))


def test_beyond_the_limit_still_sorts(kvr, oracle_mod):
    _check(kvr, oracle_mod, workloads.random_case(43, 3000, 5, 3300, 2, ties=True))


@pytest.mark.parametrize("shape", ["crowded", "heavy", "beyond", "equal_rows", "infinite_rows",
                                   "tiny_widths", "far_below", "tiny_waits",
                                   "denormal_waits", "no_inf"])
def test_extreme_samples(kvr, oracle_mod, shape):
    rng = np.random.Generator(np.random.PCG64(9))
    wl = workloads.random_case(47, 70001, 3, 40, 4, ties=True, inf_last=shape != "no_inf")
    if shape == "crowded":               # every wait in one bin, most of them equal
        wl.wait_s = np.where(rng.random(wl.n) < 0.9, 100.0, 100.0 + rng.random(wl.n))
    elif shape == "heavy":               # the largest context sizes: the limbs' carries
        wl.ctx_tokens = np.full(wl.n, 2 ** 31 - 1, dtype=np.int32)
    elif shape == "beyond":              # nearly every wait past the last finite deadline
        wl.wait_s = 1e7 * (1.0 + rng.random(wl.n))
        wl.wait_s[:5] = 1.0
    elif shape == "equal_rows":          # t1 swallows t2: runs of equal deadlines
        wl.t1 = np.array([0.0, 1e17, 2e17])
        wl.wait_s[:100] = 1e17
        wl.wait_s[100:200] = 1.5e17
    elif shape == "infinite_rows":       # finite timers whose deadlines overflow
        wl.t1 = np.array([0.0, 1e308, 1.7e308])
        wl.t2 = np.concatenate([np.geomspace(5.0, 1e5, 30), np.geomspace(1e308, 1.7e308, 9),
                                [np.inf]])
        wl.ctx_tokens = np.full(wl.n, 3, dtype=np.int32)
    elif shape == "tiny_widths":         # thresholds a denormal apart, and denormal waits
        wl.t1 = np.array([0.0, 5e-324, 1e-323])
        wl.wait_s[:1000] = rng.integers(0, 6, 1000) * 5e-324
    elif shape == "far_below":           # waits many binades below every timer
        wl.wait_s = 10.0 ** rng.uniform(-300.0, -30.0, wl.n)
    elif shape in ("tiny_waits", "denormal_waits"):
        # prices at which T*w decides the costs although every wait is far below
        # 2^-958 s: no holding price, resume prices of the size of alpha_1 * w
        unit = 1e-300 if shape == "tiny_waits" else 1e-320
        wl.wait_s = unit * (0.5 + rng.random(wl.n))
        wl.t1 = np.array([0.0, 0.8 * unit, 1.0])
        wl.lam = np.array([0.1, 0.2])
        wl.platform = dict(wl.platform, hbm_usable_bytes=wl.kv_bytes_per_token,
                           host_link_bytes_per_s=1e304, prefill_tokens_per_s=1e300)
    _check(kvr, oracle_mod, wl)


def test_domain_errors_without_an_order(kvr):
    import torch
    wl = workloads.random_case(5, 5000, 2, 20, 2)
    g = kvr.PolicyGrid(wl.t1, wl.t2, wl.lam)
    for what in ("nan", "inf", "neg", "ctx"):
        w, T = wl.wait_s.copy(), wl.ctx_tokens.copy()
        if what == "ctx":
            T[17] = 0
        else:
            w[4999] = {"nan": np.nan, "inf": np.inf, "neg": -1.0}[what]
        with pytest.raises(kvr.KvrError) as ei:
            kvr.kvr_cost_grid(_dev(w, torch.float64), _dev(T, torch.int32), _lib_prices(kvr, wl), g,
                              method=kvr.KVR_SORTED)
        assert ei.value.code == kvr.KVR_E_DOMAIN
