"""The order that the sorted method returns, at the sizes where its tiles change:
one block, tiles of 256 and 512 threads by two keys and of 1,024 by two and four
whose counts the scatter sums itself, the first and last of each, full tiles and
remainders, and the first size with a scan of its own.  An order is whole
numbers: it equals the stable order of the waits, equal waits (and zeros of both
signs) in input order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2048, 2049, 2560, 65535, 65536, 65537, 262143, 262144, 262145,
                               524288, 524289, 1048575, 1048576, 1048577])
@pytest.mark.parametrize("law", ["ties", "one", "spread"])
def test_order_is_stable(n, law):
    import torch
    import paper_2608_30830_amd as kvr
    rng = np.random.Generator(np.random.PCG64(n))
    if law == "ties":
        w = rng.integers(0, 37, n) / 8.0
        w[::5] *= -0.0
        w = np.where(w == 0, w, np.abs(w))
    elif law == "one":
        w = np.full(n, 3.5)
    else:   # every digit of the keys varies
        w = np.ldexp(1.0 + rng.random(n), rng.integers(-900, 900, n))
    T = rng.integers(1, 9, n, dtype=np.int32)
    p = kvr.kvr_prices_from_platform(131072.0, 250e9, 50e9, 2e4)
    g = kvr.PolicyGrid([0.0], [10.0, np.inf], [0.5])
    cost, perm = kvr.kvr_cost_grid(torch.as_tensor(w).cuda(), torch.as_tensor(T).cuda(), p, g,
                                   method=kvr.KVR_SORTED, want_perm=True)
    assert np.array_equal(perm.cpu().numpy(), np.argsort(w + 0.0, kind="stable"))


@pytest.mark.parametrize("n,k2", [(1048575, 3), (1048576, 512), (1048576, 513), (1048576, 2)])
def test_costs_beside_the_order(oracle_mod, n, k2):
    """From 2^20 waits and up to n / 2,048 policies the costs beside a requested
    order come from the per-bin sums, on the other side of the line from the scans of the
    sorted waits: against the oracle's closed form on both, which like them sums n
    products of one sign (1e-12 relative), with the order bit for bit."""
    import torch
    import paper_2608_30830_amd as kvr
    rng = np.random.Generator(np.random.PCG64(n + k2))
    w, T = rng.exponential(1800.0, n), rng.integers(1, 40000, n, dtype=np.int32)
    p = kvr.kvr_prices_from_platform(131072.0, 250e9, 50e9, 2e4)
    t2, lam = np.append(np.geomspace(5.0, 90000.0, k2 - 1), np.inf), np.array([0.2, 0.9])
    g = kvr.PolicyGrid([0.0], t2, lam)
    cost, perm = kvr.kvr_cost_grid(torch.as_tensor(w).cuda(), torch.as_tensor(T).cuda(), p, g,
                                   method=kvr.KVR_SORTED, want_perm=True)
    ref = oracle_mod.closed_form_grid(w, T, oracle_mod.prices_from_platform(131072.0, 250e9, 50e9, 2e4),
                                      np.zeros(1), t2, lam)
    assert np.all(np.abs(cost.cpu().numpy() - ref) <= 1e-12 * np.abs(ref))
    assert np.array_equal(perm.cpu().numpy(), np.argsort(w, kind="stable"))
