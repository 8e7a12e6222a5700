"""Sweeps that may fill the device, enqueued together on several streams:
replays of captured books, eager books and single options run one after
another and each gives its own prices."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KW = dict(S0=100.0, r=0.04, sigma=0.3, T=1.0)


def _book(amq, lo, n_paths, n_dates, n):
    return amq.make_options([dict(KW, K=lo + q, is_call=q % 2 == 1, n_paths=n_paths + 37 * q, n_dates=n_dates)
                             for q in range(n)])


@pytest.mark.parametrize("dtype", ["fp32", "fp64"])
def test_replays_and_eager_calls_on_several_streams(dtype):
    import torch
    import paper_1205_0106_amd as amq
    assert torch.cuda.is_available()
    b = amq.make_basis("monomial", 2)
    # options of many tiles, so that a grid kept half resident could not go on
    books = [_book(amq, 90.0, 1 << 20, 5, 6), _book(amq, 95.0, 700000, 7, 8)]
    eager = _book(amq, 99.0, 900000, 6, 5)
    one = amq.make_params(**KW, K=101.0)
    streams = [torch.cuda.Stream() for _ in range(4)]
    pr, single = amq.Pricer(0, stream=streams[2]), amq.Pricer(0, stream=streams[3])
    want = [amq.Pricer(0).price_batch(o, b, dtype) for o in books]
    want_eager, want_one = pr.price_batch(eager, b, dtype), single.price(one, 1 << 20, 8, b, dtype)
    ws = [torch.empty(amq.am_batch_workspace_bytes(o, b, dtype), dtype=torch.uint8, device="cuda") for o in books]
    graphs = [amq.BatchGraph(o, b, dtype, w) for o, w in zip(books, ws)]
    torch.cuda.synchronize()
    for turn in range(4):
        print(f"  turn {turn} {dtype}", flush=True)
        graphs[0].launch(streams[0])
        graphs[1].launch(streams[1])
        single.price(one, 1 << 20, 8, b, dtype, wait=False)
        got_eager = pr.price_batch(eager, b, dtype)
        graphs[1].launch(streams[0])
        graphs[0].launch(streams[1])
        got_one = single.price(one, 1 << 20, 8, b, dtype)
        assert np.array_equal(got_eager, want_eager) and got_one == want_one
        for g, w in zip(graphs, want):
            assert np.array_equal(g.results(), w)
    for g in graphs:
        g.close()


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
