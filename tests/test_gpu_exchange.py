"""The per-date device-wide sum at the edges of its forms: one wave spinning
on every group's row (at most 512 row words: 32 groups of 16-word rows, 16 of
32-word rows), and the arrival counters above."""
import pytest

pytestmark = pytest.mark.gpu

# f64 tiles of 512 threads x 2 paths: 1024 paths a group
TILE = 1024
# The GPU's sums and solve and the oracle's Givens QR round differently (1e-16
# relative each, amplified by the standardised design's condition number, below
# 1e4 for these bases): 1e-9 of a price of order 5 leaves two decades.
TOL = 5e-9


@pytest.mark.parametrize("groups,degree", [(1, 2), (4, 2), (5, 3), (16, 4), (17, 2), (32, 4), (33, 2), (1, 5), (8, 5),
                                           (9, 6), (16, 5), (17, 5)])
@pytest.mark.parametrize("ragged", [0, 37])
def test_row_exchange_edges(orc, groups, degree, ragged):
    import torch
    import paper_1205_0106_amd as amq
    assert torch.cuda.is_available()
    pr = amq.Pricer(0)
    kw = dict(S0=36.0, K=40.0, r=0.06, sigma=0.2, T=1.0)
    N, M = groups * TILE - ragged, 6
    p, b = amq.make_params(**kw), amq.make_basis("monomial", degree)
    print(f"  exchange: groups={groups} degree={degree} N={N}", flush=True)
    amq.am_debug_set_sweep_tile(512, 2)
    try:
        price, se = pr.price(p, N, M, b, "fp64")
        again = pr.price(p, N, M, b, "fp64")
    finally:
        amq.am_debug_set_sweep_tile(0, 0)
    assert again == (price, se)
    want = orc.price_american(**kw, N=N, M=M, kind=orc.MONOMIAL, degree=degree)
    assert abs(price - want.price) <= TOL
    # group 0's record: every date solved, stamps in order
    rec = pr.views(N, M, b, "fp64")["rec"].cpu().numpy()
    for k in range(1, M):
        assert rec[k, 8] == 1.0 and 0 < rec[k, 36] <= rec[k, 32] <= rec[k, 33] <= rec[k, 34]


# 512-thread register-resident tiles are compiled apart for few groups and for
# more; 256-thread ones hold every form.  The two differ in the order of their
# sums only: 1e-16 relative each, amplified by a condition number below 1e4, in a
# price of order 10.
@pytest.mark.parametrize("dtype,ppt", [("fp32", 4), ("fp64", 2)])
@pytest.mark.parametrize("basis,degree,groups", [("monomial", 1, 32), ("monomial", 2, 33), ("monomial", 4, 32), ("monomial", 4, 33),
                                                 ("monomial", 5, 16), ("monomial", 5, 17), ("laguerre", 3, 9),
                                                 ("laguerre", 3, 32), ("laguerre", 3, 33), ("laguerre", 3, 200)])
def test_few_and_more_groups(dtype, ppt, basis, degree, groups):
    import torch
    import paper_1205_0106_amd as amq
    assert torch.cuda.is_available()
    pr = amq.Pricer(0)
    p, b = amq.make_params(S0=100.0, K=102.0, r=0.05, sigma=0.3, T=1.0, is_call=False), amq.make_basis(basis, degree)
    N, M = groups * 512 * ppt - 3, 7
    print(f"  exchange: {dtype} {basis} {degree} groups={groups}", flush=True)
    got = {}
    for wg in (512, 256):
        amq.am_debug_set_sweep_tile(wg, ppt)
        try:
            got[wg] = pr.price(p, N, M, b, dtype)
        finally:
            amq.am_debug_set_sweep_tile(0, 0)
    assert abs(got[512][0] - got[256][0]) <= 1e-10 and abs(got[512][1] - got[256][1]) <= 1e-10


# groups dealt to several XCDs (stride 3: all eight in turn; 4: two): they find
# that the others announced another one and exchange through memory.  The same
# sums in the same order.
@pytest.mark.parametrize("stride", [2, 3, 4, 7])
@pytest.mark.parametrize("dtype,ppt,basis,degree,groups", [("fp64", 2, "monomial", 2, 2), ("fp64", 2, "monomial", 4, 17),
                                                           ("fp64", 2, "monomial", 2, 32), ("fp64", 2, "laguerre", 3, 9),
                                                           ("fp64", 2, "monomial", 5, 16), ("fp32", 4, "monomial", 2, 25)])
def test_groups_on_several_xcds(stride, dtype, ppt, basis, degree, groups):
    import torch
    import paper_1205_0106_amd as amq
    assert torch.cuda.is_available()
    pr = amq.Pricer(0)
    p, b = amq.make_params(S0=100.0, K=102.0, r=0.05, sigma=0.3, T=1.0, is_call=False), amq.make_basis(basis, degree)
    N, M = groups * 512 * ppt - 3, 25
    print(f"  exchange: stride={stride} {dtype} {basis} {degree} groups={groups}", flush=True)
    amq.am_debug_set_sweep_tile(512, ppt)
    try:
        want = pr.price(p, N, M, b, dtype)
        amq.am_debug_set_group_stride(stride)
        for _ in range(3):
            assert pr.price(p, N, M, b, dtype) == want
    finally:
        amq.am_debug_set_group_stride(0)
        amq.am_debug_set_sweep_tile(0, 0)
