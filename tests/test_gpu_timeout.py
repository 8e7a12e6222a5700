"""A bounded wait that runs out in a book (forced from the host by a tiny
limit): every workgroup exits and no option that was not priced reads as
priced, in books of both storage types too."""
import time

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,large_tile", [("fp32", True), ("fp32", False), ("fp64", True)])
def test_no_unpriced_option_is_ok(dtype, large_tile):
    import torch
    import paper_1205_0106_amd as amq
    assert torch.cuda.is_available()
    kw = dict(S0=100.0, r=0.04, sigma=0.3, T=1.0, is_call=False)
    # more tiles than the device holds, those of few dates claimed last; in
    # binary32 requests the small options are stored in binary64
    n_big = 48 if large_tile else 12
    specs = [dict(kw, K=100.0 + q, n_paths=262144, n_dates=6) for q in range(n_big)]
    specs += [dict(kw, K=90.0 + q, n_paths=12000, n_dates=3) for q in range(40)]
    b = amq.make_basis("monomial", 2)
    opts = amq.make_options(specs)
    first = amq.make_options([dict(kw, K=100.0, n_paths=1 << 19, n_dates=100)])
    want = None   # the same server's results where no wait runs out
    for limit in (0, 1):
        print(f"  book under spin limit {limit}: {dtype} large_tile={large_tile}", flush=True)
        amq.am_debug_set_spin_limit(limit)
        try:
            srv = amq.Server(3 << 30, b, dtype, n_streams=1, max_batch_requests=128, max_batch_path_steps=1e12,
                             large_tile=large_tile)
        finally:
            amq.am_debug_set_spin_limit(0)
        got = {}
        with srv:
            srv.submit(first[0], 1000)   # holds the device while the others queue up
            for i in range(len(specs)):
                srv.submit(opts[i], i)
            t0 = time.time()
            while len(got) < len(specs) + 1:
                for r in srv.poll():
                    got[r["id"]] = r
                assert time.time() - t0 < 60.0
                time.sleep(0.001)
        late = sum(r["status"] == amq.AM_ETIMEOUT for r in got.values())
        print(f"  {late} of {len(got)} timed out", flush=True)
        assert limit or late == 0
        res = [(got[i]["price"], got[i]["std_err"]) for i in range(len(specs))]
        if want is None:
            want = res
        for i in range(len(specs)):
            assert got[i]["status"] == amq.AM_ETIMEOUT or (got[i]["status"] == amq.AM_OK and res[i] == want[i]), i
