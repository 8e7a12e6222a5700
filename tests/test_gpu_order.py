"""Sweeps that may fill the device, enqueued together on several streams, run
one after another and each gives its own prices."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KW = dict(S0=100.0, r=0.04, sigma=0.3, T=1.0)


def _book(amq, lo, n_paths, n_dates, n):
    return amq.make_options([dict(KW, K=lo + q, is_call=q % 2 == 1, n_paths=n_paths + 37 * q, n_dates=n_dates)
                             for q in range(n)])


def test_call_captured_by_the_caller():
    import torch
    import paper_1205_0106_amd as amq
    assert torch.cuda.is_available()
    b, p = amq.make_basis("monomial", 2), amq.make_params(**KW, K=100.0)
    N, M = 50001, 12
    s, other = torch.cuda.Stream(), torch.cuda.Stream()
    pr, pb = amq.Pricer(0, stream=s), amq.Pricer(0, stream=other)
    book = _book(amq, 95.0, 20000, 9, 4)
    want_book = pb.price_batch(book, b, "fp64")
    want = pr.price(p, N, M, b, "fp64")          # schedule and workspace are set up here
    want_book = pb.price_batch(book, b, "fp64")  # (the last sweep was on another stream)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        pr.price(p, N, M, b, "fp64", wait=False)
    result = pr.views(N, M, b, "fp64")["result"]
    for turn in range(3):
        print(f"  replay {turn}", flush=True)
        # eager calls on other streams go on as before
        assert np.array_equal(pb.price_batch(book, b, "fp64"), want_book)
        result.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert tuple(result[:2].tolist()) == want
    assert pr.price(p, N, M, b, "fp64") == want
