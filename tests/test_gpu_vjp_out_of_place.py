"""The backward's sweeps that read one state and write the next: a hub row of
3,000 entries in pieces, rows of every lane count, rows whose weights are all
zero and rows without entries (both keep their vector), by launches and by one
launch for all colours (the same bits), stored and rebuilt, against the FP64
oracle (float32 states, gradients within 1e-4 of the largest component: 30
times the rounding of 5 sweeps of float32 averages)."""
import numpy as np
import pytest

from oracle import oracle as O
from workloads import graphs as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _graph():
    n = 3001
    v = np.arange(1, n)
    rng = np.random.default_rng(4)
    chords = rng.integers(1, n, (4000, 2))
    chords = np.unique(np.sort(chords, axis=1), axis=0)
    chords = chords[chords[:, 1] - chords[:, 0] > 1]
    chords = chords[~((chords[:, 0] == 1) & (chords[:, 1] == n - 1))]
    # rows n .. n + 9 hang on nodes 1 .. 10 by zero weights, the next 3 are alone
    u = np.concatenate([np.zeros(n - 1, np.int64), v[:-1], chords[:, 0], np.arange(1, 11)])
    t = np.concatenate([v, v[1:], chords[:, 1], n + np.arange(10)])
    w = rng.uniform(0.5, 2.0, u.size).astype(np.float32)
    w[-10:] = 0.0
    return W.csr_from_edges(n + 13, u, t, w, "hub")


@pytest.mark.parametrize("K", [4, 16, 64])
def test_out_of_place_sweeps(K, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_08942_amd import graphreduce as G

    g = _graph()
    c, nc = O.colour_greedy(g.n, g.row_ptr, g.col, 9, False)
    rng = np.random.default_rng(K)
    X0 = O.init_vectors(g.n, K, 31).astype(np.float32)
    Gc = rng.standard_normal((g.n, K)).astype(np.float32)
    dev = "cuda:0"
    dg = G.DeviceGraph.from_numpy(g.row_ptr, g.col, g.w, dev)
    el = G.gr_edge_list(dg)
    cd = torch.from_numpy(np.asarray(c, np.int32)).to(dev)
    eoe, eu, ev = O.edge_index(g.n, g.row_ptr, g.col)
    wE = np.zeros(eu.size)
    wE[eoe] = g.w
    for S in (1, 2, 5):
        rgw, rgX = O.smooth_vjp(g.n, g.row_ptr, g.col, wE, c, nc, X0.astype(np.float64),
                                Gc.astype(np.float64), S)
        first = None
        for flow in ("0", "1"):
            for store in (True, False):
                print(f"[gpu-case] out of place K={K} S={S} flow={flow} store={store}", flush=True)
                monkeypatch.setenv("GR_GS_FLOW", flow)
                gw, gX = G.gr_smooth_vjp(dg, el, cd, nc, torch.from_numpy(X0).to(dev),
                                         torch.from_numpy(Gc).to(dev), S, store)
                if first is None:
                    first = (gw, gX)
                    hw, hX = gw.cpu().numpy(), gX.cpu().numpy()
                    assert np.max(np.abs(hw - rgw)) <= 1e-4 * np.max(np.abs(rgw))
                    assert np.max(np.abs(hX - rgX)) <= 1e-4 * np.max(np.abs(rgX))
                assert torch.equal(gw, first[0]) and torch.equal(gX, first[1])
