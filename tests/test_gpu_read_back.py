"""Sizes and flags read back through pinned pages: a transfer that does not fit
a page (more than 800 colours), and more threads at once than there are
pages, each on a stream and a workspace of its own."""
import threading

import numpy as np
import pytest

from oracle import oracle as O
from workloads import graphs as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_08942_amd import graphreduce as G

    return G


def test_more_than_a_page():
    G = _G()
    g = W.complete(900)
    print("[gpu-case] 900 colours", flush=True)
    dg = G.DeviceGraph.from_numpy(g.row_ptr, g.col, g.w, "cuda:0")
    colours, nc = G.gr_colour_greedy(dg, 3)
    assert nc == 900
    X = G.gr_init_vectors(g.n, 4, 5, "f32", "cuda:0")
    X0 = X.cpu().numpy()
    G.gr_smooth(dg, colours, nc, X, 1)
    ref = O.smooth(g.n, g.row_ptr, g.col, g.w.astype(np.float64), colours.cpu().numpy(), nc, X0, 1)
    # float32 sums of 899 terms of magnitude below max|X0|
    assert np.abs(X.cpu().numpy() - ref).max() <= 899 * 2.0**-24 * np.abs(X0).max()


@pytest.mark.parametrize("bad", [-1, 2])
def test_a_bad_colour_is_still_refused(bad):
    G = _G()
    g = W.grid2d(20, 20)
    dg = G.DeviceGraph.from_numpy(g.row_ptr, g.col, g.w, "cuda:0")
    X = G.gr_init_vectors(g.n, 4, 5, "f32", "cuda:0")
    for where, value in ((17, bad), (17, 1 - g.colours[17])):
        c = g.colours.copy()
        c[where] = value
        with pytest.raises(G.GraphReduceError) as e:
            G.gr_smooth(dg, torch.from_numpy(c).to("cuda:0"), 2, X, 1)
        assert e.value.code == -3


def test_more_threads_than_pages():
    G = _G()
    g = W.knn2d(1500, 8, seed=4)
    dg = G.DeviceGraph.from_numpy(g.row_ptr, g.col, g.w, "cuda:0")
    want = G.gr_reduce(dg, 4, 2, 8.0, 1, 2)
    want = (want.agg.clone(), want.coarse.col.clone(), want.coarse.w.clone())
    torch.cuda.synchronize()
    wrong = []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                ws = torch.empty(G.gr_workspace_size(g.n, g.nnz, 4), dtype=torch.uint8,
                                 device="cuda:0")
                for _ in range(3):
                    r = G.gr_reduce(dg, 4, 2, 8.0, 1, 2, ws=ws)
                torch.cuda.current_stream().synchronize()
                for a, b in zip((r.agg, r.coarse.col, r.coarse.w), want):
                    if not torch.equal(a, b):
                        wrong.append(k)
        except Exception as e:  # told by the main thread
            wrong.append((k, repr(e)))

    print("[gpu-case] 20 threads", flush=True)
    threads = [threading.Thread(target=work, args=(k,)) for k in range(20)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong
