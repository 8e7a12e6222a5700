"""Slab tiles (one to four units per group) at the edges of their split:
single options forced onto them, and books, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KW = dict(S0=100.0, r=0.04, sigma=0.3, T=1.5)
# binary64: the kernels' sums and the oracle's QR round differently by 1e-16
# relative, amplified by the design's condition number (below 1e4): 1e-9 of a
# price of order 10.  binary32 storage is compared with the oracle on the same
# storage: a cashflow that rounds the other way moves 6e-8 of one path of
# 20000 and more, and near-ties in the exercise test at most one decision of
# value 1 each: 1e-4.
TOL = {"fp64": 1e-8, "fp32": 1e-4}


@pytest.fixture(scope="module")
def pricer():
    import torch
    import paper_1205_0106_amd as amq
    assert torch.cuda.is_available()
    return amq.Pricer(0)


# units: 4096 binary64 or 8192 binary32 paths of 512-thread groups
@pytest.mark.parametrize("dtype,ppt,N", [("fp64", 32, 4), ("fp64", 32, 4095), ("fp64", 32, 4097), ("fp64", 32, 12289),
                                         ("fp64", 32, 40000), ("fp32", 64, 16384), ("fp32", 64, 24577),
                                         ("fp32", 64, 65535)])
@pytest.mark.parametrize("degree,call", [(1, True), (2, False), (4, True)])
def test_single_option_units(orc, pricer, dtype, ppt, N, degree, call):
    import paper_1205_0106_amd as amq
    if N < degree + 2:
        pytest.skip("fewer paths than the basis takes")
    M, K = 9, 96.0 if call else 104.0
    p, b = amq.make_params(**KW, K=K, is_call=call), amq.make_basis("monomial", degree)
    print(f"  slab: {dtype} N={N} d={degree} call={call}", flush=True)
    amq.am_debug_set_sweep_tile(512, ppt)
    try:
        price, se = pricer.price(p, N, M, b, dtype)
    finally:
        amq.am_debug_set_sweep_tile(0, 0)
    want = orc.price_american(**KW, K=K, N=N, M=M, kind=orc.MONOMIAL, degree=degree, is_call=call,
                              store32=dtype == "fp32")
    assert abs(price - want.price) <= TOL[dtype]
    assert abs(se - want.std_err) <= TOL[dtype]
    pv = pricer.views(N, M, b, dtype)["PV"].double().cpu().numpy()
    assert abs(pv.mean() - want.price) <= TOL[dtype]     # every path's cashflow written, each once


# 256-thread groups in books: units of 4096 binary32 or 2048 binary64 paths
@pytest.mark.parametrize("dtype,sizes", [("fp64", [100, 2047, 2048, 2049, 6145, 8192, 8193, 20481]),
                                         ("fp32", [16384, 16385, 20480, 20481, 32768, 36865])])
def test_book_units(orc, pricer, dtype, sizes):
    import paper_1205_0106_amd as amq
    specs = [dict(KW, K=90.0 + 3 * q, is_call=bool(q % 2), n_paths=n, n_dates=5 + q) for q, n in enumerate(sizes)]
    got = pricer.price_batch(amq.make_options(specs), amq.make_basis("monomial", 2), dtype)
    for q, d in enumerate(specs):
        want = orc.price_american(**KW, K=d["K"], N=d["n_paths"], M=d["n_dates"], kind=orc.MONOMIAL, degree=2,
                                  is_call=d["is_call"], store32=dtype == "fp32")
        assert abs(got[q, 0] - want.price) <= TOL[dtype], (q, d)


def test_mixed_storage_book(orc, pricer):
    # a binary32 request whose options straddle the storage floor prices both
    # kinds in one sweep: each option as in a book of its own kind, bit for bit
    import paper_1205_0106_amd as amq
    sizes = [16384, 40000, 16383, 300, 20481, 9000, 65536, 5]
    specs = [dict(KW, K=92.0 + 2 * q, is_call=bool(q % 3 == 0), n_paths=n, n_dates=4 + 3 * q)
             for q, n in enumerate(sizes)]
    for degree in (2, 3):
        b = amq.make_basis("monomial", degree)
        got = pricer.price_batch(amq.make_options(specs), b, "fp32")
        for big in (True, False):
            idx = [q for q, n in enumerate(sizes) if (n >= 16384) == big]
            alone = pricer.price_batch(amq.make_options([specs[q] for q in idx]), b, "fp32")
            assert np.array_equal(got[idx], alone)
        want = orc.price_american(**KW, K=specs[2]["K"], N=sizes[2], M=specs[2]["n_dates"], kind=orc.MONOMIAL,
                                  degree=degree, is_call=specs[2]["is_call"])
        assert abs(got[2, 0] - want.price) <= TOL["fp64"]


# one unit a group: just past the rows that one wave reads whole (32 groups of
# 16-word rows, 16 of 32-word ones), uneven and even teams, the most relayed
@pytest.mark.parametrize("groups,degree", [(33, 2), (40, 3), (64, 2), (255, 1), (256, 2), (17, 5), (33, 6)])
def test_relayed_sum(orc, pricer, groups, degree):
    import paper_1205_0106_amd as amq
    N, M, K = groups * 4096 - 11, 4, 103.0
    p, b = amq.make_params(**KW, K=K, is_call=False), amq.make_basis("monomial", degree)
    print(f"  relay: groups={groups} d={degree}", flush=True)
    amq.am_debug_set_sweep_tile(512, 32)
    try:
        price, se = pricer.price(p, N, M, b, "fp64")
        assert pricer.price(p, N, M, b, "fp64") == (price, se)
    finally:
        amq.am_debug_set_sweep_tile(0, 0)
    want = orc.price_american(**KW, K=K, N=N, M=M, kind=orc.MONOMIAL, degree=degree)
    assert abs(price - want.price) <= TOL["fp64"]
    assert abs(se - want.std_err) <= TOL["fp64"]
