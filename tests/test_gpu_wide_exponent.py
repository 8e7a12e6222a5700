"""Log-prices beyond the narrow exponent, to arguments far past the range in
which exp is finite and nonzero."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# sigma sqrt(T) from 10 to 10^6: drifts -sigma^2 T / 2 to -5e11, through the
# arguments at which 64 x / ln 2 leaves 32 bits (2.3e7, and its multiples); and
# rates that take every path to infinity
@pytest.mark.parametrize("sigma,r", [(10.0, 0.03), (6700.0, 0.03), (6900.0, 0.03), (8000.0, 0.03), (9600.0, 0.03),
                                     (9700.0, 0.03), (1.2e4, 0.03), (3e4, 0.03), (1e6, 0.03), (0.5, 4e7), (0.5, 1.2e8)])
@pytest.mark.parametrize("dtype", ["fp64", "fp32"])
def test_paths_at_extreme_arguments(orc, sigma, r, dtype):
    import torch
    import paper_1205_0106_amd as amq
    assert torch.cuda.is_available()
    N, M = 1024 if dtype == "fp64" else 16384 + 3, 5
    kw = dict(S0=100.0, K=100.0, r=r, sigma=sigma, T=1.0)
    print(f"  wide exponent: sigma={sigma} r={r} {dtype}", flush=True)
    got = np.asarray(amq.am_debug_generate(0, amq.make_params(**kw), N, M, dtype))
    want = np.asarray(orc.paths(**kw, N=N, M=M))
    if dtype == "fp32":
        with np.errstate(over="ignore", under="ignore"):
            want = want.astype(np.float32).astype(np.float64)
    assert np.array_equal(np.isinf(got), np.isinf(want)) and not np.isnan(got).any()
    assert np.array_equal(got == 0.0, want == 0.0)
    # a put that no path leaves in the money for long, not exercised early: the
    # discounted strike where every path ends at 0
    if sigma >= 6700.0:
        p = amq.make_params(**kw, is_call=False, allow_exercise=False)
        price, se = amq.am_price_american(p, N, M, amq.make_basis("monomial", 2), dtype)
        assert abs(price - 100.0 * math.exp(-0.03)) <= (1e-12 if dtype == "fp64" else 1e-5) and se <= 1e-6
