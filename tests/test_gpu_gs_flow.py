"""All sweeps of a smoothing in one launch, rows waiting for their neighbours'
values, give the same bits as one launch per colour step: tiers of every
width, split hub rows, isolated rows, rows whose weights are all zero, one
sweep and several, NaNs whose bits are all ones; and a wait that runs out
(forced from the host) ends in the launches' result."""
import numpy as np
import pytest

from oracle import oracle as O
from workloads import graphs as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _graphs():
    m = 60  # left rows with 1 .. 60 entries; right row 0 has only zero weights
    u, v = np.nonzero(np.tril(np.ones((m, m))))
    w = np.random.default_rng(5).uniform(0.5, 2.0, u.size).astype(np.float32)
    w[v == 0] = 0.0
    return {
        "degrees": W.csr_from_edges(2 * m, u, v + m, w),
        "hubs": W.chung_lu(10000, mean_deg=700.0, seed=7),
        "isolated": W.with_isolated(W.random_weighted(40, 0.15, seed=9), 3),
        "knn": W.knn2d(3000, 10, seed=2),
    }


def _bits(X):
    return X.view(torch.int16 if X.dtype == torch.bfloat16 else torch.int32).cpu().numpy()


@pytest.mark.parametrize("dtype,K", [("f32", 4), ("f32", 16), ("f32", 64), ("bf16", 8),
                                     ("bf16", 64)])
def test_flow_gives_the_launches_bits(dtype, K, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_08942_amd import graphreduce as G

    for name, g in _graphs().items():
        c, nc = O.colour_greedy(g.n, g.row_ptr, g.col, 3, False)
        colours = torch.from_numpy(np.asarray(c, np.int32)).to("cuda:0")
        dg = G.DeviceGraph.from_numpy(g.row_ptr, g.col, g.w, "cuda:0")
        X0 = torch.from_numpy(O.init_vectors(g.n, K, 17).astype(np.float32)).to("cuda:0").to(
            torch.float32 if dtype == "f32" else torch.bfloat16).contiguous()
        for sweeps in (1, 2, 5):
            out = {}
            for mode in ("0", "1", "limit"):
                print(f"[gpu-case] flow {name} K={K} {dtype} sweeps={sweeps} {mode}", flush=True)
                monkeypatch.setenv("GR_GS_FLOW", "0" if mode == "0" else "1")
                if mode == "limit":
                    monkeypatch.setenv("GR_GS_SPIN_LIMIT", "1")
                X = X0.clone()
                G.gr_smooth(dg, colours, nc, X, sweeps)
                torch.cuda.synchronize()
                out[mode] = _bits(X)
                monkeypatch.delenv("GR_GS_SPIN_LIMIT", raising=False)
            monkeypatch.delenv("GR_GS_FLOW")
            assert np.array_equal(out["0"], out["1"]), (name, sweeps)
            assert np.array_equal(out["0"], out["limit"]), (name, sweeps)


def test_flow_passes_nans_on(monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_08942_amd import graphreduce as G

    g = W.knn2d(3000, 10, seed=2)
    c, nc = O.colour_greedy(g.n, g.row_ptr, g.col, 3, False)
    colours = torch.from_numpy(np.asarray(c, np.int32)).to("cuda:0")
    dg = G.DeviceGraph.from_numpy(g.row_ptr, g.col, g.w, "cuda:0")
    X0 = O.init_vectors(g.n, 16, 17).astype(np.float32)
    X0.view(np.uint32)[::500, :] = 0xFFFFFFFF
    X0[7, 3] = np.inf
    out = {}
    for mode in ("0", "1"):
        print(f"[gpu-case] flow NaN {mode}", flush=True)
        monkeypatch.setenv("GR_GS_FLOW", mode)
        X = torch.from_numpy(X0).to("cuda:0")
        G.gr_smooth(dg, colours, nc, X, 2)
        out[mode] = X.cpu().numpy()
    assert np.isnan(out["0"]).any()
    assert np.array_equal(out["0"], out["1"], equal_nan=True)
