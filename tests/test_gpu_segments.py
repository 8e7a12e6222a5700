"""Path generation in schedule segments (few path blocks) against whole
schedules (many): the same paths bit for bit, plain and digitally shifted."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KW = dict(S0=100.0, K=105.0, r=0.03, sigma=0.35, T=1.5)
MANY = 4096 * 64 + 37   # enough blocks that schedules up to 280 dates stay whole


@pytest.fixture(scope="module")
def pricer():
    import torch
    import paper_1205_0106_amd as amq
    assert torch.cuda.is_available()
    return amq.Pricer(0)


# below, at and past the date counts where 2, 4 and 8 segments begin; chunk
# remainders of every size; more dates than one segment's tables hold
@pytest.mark.parametrize("M", [1, 2, 7, 15, 16, 17, 31, 32, 33, 63, 64, 65, 67, 100, 280, 281, 365, 640])
@pytest.mark.parametrize("dtype", ["fp64", "fp32"])
def test_segments_give_the_same_paths(pricer, M, dtype):
    import paper_1205_0106_amd as amq
    few = 16384 + 5 if dtype == "fp32" else 1000 + 5
    b, p = amq.make_basis("monomial", 2), amq.make_params(**KW)
    print(f"  segments: M={M} {dtype} N={few} and {MANY}", flush=True)
    pricer.price(p, few, M, b, dtype)
    got = pricer.views(few, M, b, dtype)["S"].clone()
    pricer.price(p, MANY, M, b, dtype)
    want = pricer.views(MANY, M, b, dtype)["S"][:, :few]
    assert np.array_equal(got.cpu().numpy(), want.cpu().numpy())


def test_batch_segments_equal_the_option_in_a_large_book(pricer):
    # a few options price in segments, the same ones among many in whole schedules
    import paper_1205_0106_amd as amq
    opt = dict(S0=100.0, K=97.0, r=0.04, sigma=0.3, T=1.0, is_call=True, n_paths=17000, n_dates=75)
    big = [dict(opt, n_paths=30000 + q, n_dates=20) for q in range(12)]
    b = amq.make_basis("monomial", 2)
    for dtype in ("fp32", "fp64"):
        alone = pricer.price_batch(amq.make_options([opt]), b, dtype)
        mixed = pricer.price_batch(amq.make_options(big + [opt]), b, dtype)
        assert np.array_equal(np.asarray(alone)[0], np.asarray(mixed)[-1])


@pytest.mark.parametrize("sigma,T,r", [(3.0, 100.0, 4.5), (20.0, 36.0, 200.0)])
def test_paths_beyond_the_narrow_exponent(orc, pricer, sigma, T, r):
    # deviations so large that log-prices may leave +-700: the exponential's
    # general form.  The argument carries about 2e-16 of its terms (up to 10^4:
    # drift and deviation cancel) from each of the five bridge levels on either
    # side: 1e-11 relative on what is finite and normal
    import paper_1205_0106_amd as amq
    N, M = 2048, 16
    kw = dict(S0=100.0, K=100.0, r=r, sigma=sigma, T=T)
    got = np.asarray(amq.am_debug_generate(0, amq.make_params(**kw), N, M, "fp64"))
    want = np.asarray(orc.paths(**kw, N=N, M=M))
    ok = np.isfinite(want) & (want > 1e-300)
    assert ok.mean() > 0.5
    assert np.all(np.abs(got[ok] / want[ok] - 1.0) <= 1e-11)
    assert np.array_equal(np.isinf(got), np.isinf(want))


# the longest schedule whose tables let four generation groups share a CU's LDS
# stays whole in a launch of many blocks, the next one is split; so are the
# longest halves (521 dates) and the next (522, 523)
@pytest.mark.parametrize("M", [261, 262, 520, 521, 522, 523])
def test_segments_around_the_longest(pricer, M):
    import paper_1205_0106_amd as amq
    b, p = amq.make_basis("monomial", 2), amq.make_params(**KW)
    few = 1000 + 5
    print(f"  segments: M={M} N={few} and {MANY}", flush=True)
    pricer.price(p, few, M, b, "fp64")
    got = pricer.views(few, M, b, "fp64")["S"].clone()
    pricer.price(p, MANY, M, b, "fp64")
    want = pricer.views(MANY, M, b, "fp64")["S"][:, :few]
    assert np.array_equal(got.cpu().numpy(), want.cpu().numpy())
