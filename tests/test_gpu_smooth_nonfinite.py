"""Smoothing where a row's own vector is not finite: a row with weight takes the
mean of its neighbours, so its own values do not enter.  Rows of up to 32
entries, of every degree, against the FP64 oracle; launch by launch and in one
launch."""
import numpy as np
import pytest

from oracle import oracle as O
from workloads import graphs as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("flow", ["0", "1"])
@pytest.mark.parametrize("K,dtype", [(4, "f32"), (16, "f32"), (64, "f32"), (8, "bf16"),
                                     (32, "bf16")])
def test_own_vector_does_not_enter(K, dtype, flow, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_08942_amd import graphreduce as G

    m = 32
    u, v = np.nonzero(np.tril(np.ones((m, m))))  # left u has u + 1 entries, right v m - v
    w = np.random.default_rng(3).uniform(0.5, 2.0, u.size).astype(np.float32)
    g = W.csr_from_edges(2 * m, u, v + m, w)
    colours = (np.arange(2 * m) >= m).astype(np.int32)
    X = torch.from_numpy(O.init_vectors(g.n, K, 7).astype(np.float32)).to("cuda:0")
    if dtype == "bf16":
        X = X.to(torch.bfloat16)
    # the left rows come first and read right rows only
    X[0:m:3] = float("inf")
    X[1:m:3] = float("nan")
    X[2:m:3, ::2] = float("-inf")
    X0 = X.float().cpu().numpy()
    print(f"[gpu-case] own vector not finite, K={K} {dtype} flow={flow}", flush=True)
    monkeypatch.setenv("GR_GS_FLOW", flow)
    dg = G.DeviceGraph.from_numpy(g.row_ptr, g.col, g.w, "cuda:0")
    G.gr_smooth(dg, torch.from_numpy(colours).to("cuda:0"), 2, X, 1)
    got = X.float().cpu().numpy()
    assert np.isfinite(got).all()
    ref = O.smooth(g.n, g.row_ptr, g.col, g.w.astype(np.float64), colours, 2, X0, 1,
                   bf16=(dtype == "bf16"))
    # float32 sums of at most 32 terms in two steps, of values up to the
    # largest right one; bfloat16: a rounding may land on a neighbouring value
    # in either step, 2^-8 of the value to each side of the exact one
    top = np.abs(X0[m:]).max()
    tol = 2 * 32 * 2.0**-24 * top if dtype == "f32" else 2 * 2.0**-7 * top
    assert np.abs(got - ref).max() <= tol
