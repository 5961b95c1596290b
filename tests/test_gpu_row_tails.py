"""Smoothing of rows of every degree around the kernel's rounds, against the
FP64 oracle: a bipartite graph whose left rows have 1, 2, .. 70 entries (each
lane count of the degree tiers, rounds that are full and rounds with a tail)
and whose right rows then have every degree too."""
import numpy as np
import pytest

from oracle import oracle as O
from workloads import graphs as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("K,dtype", [(4, "f32"), (16, "f32"), (64, "f32"), (8, "bf16"),
                                     (32, "bf16")])
def test_smooth_every_degree(K, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_08942_amd import graphreduce as G

    m = 70
    u, v = np.nonzero(np.tril(np.ones((m, m))))  # left u has u + 1 entries
    rng = np.random.default_rng(3)
    w = rng.uniform(0.5, 2.0, u.size).astype(np.float32)
    g = W.csr_from_edges(2 * m, u, v + m, w)
    colours = (np.arange(2 * m) >= m).astype(np.int32)
    X0 = O.init_vectors(g.n, K, 7).astype(np.float32)
    X = torch.from_numpy(X0).to("cuda:0")
    if dtype == "bf16":
        X = X.to(torch.bfloat16)
        X0 = X.float().cpu().numpy()
    print(f"[gpu-case] every degree, K={K} {dtype}", flush=True)
    dg = G.DeviceGraph.from_numpy(g.row_ptr, g.col, g.w, "cuda:0")
    G.gr_smooth(dg, torch.from_numpy(colours).to("cuda:0"), 2, X, 3)
    ref = O.smooth(g.n, g.row_ptr, g.col, g.w.astype(np.float64), colours, 2, X0, 3,
                   bf16=(dtype == "bf16"))
    # float32 sums of at most 70 terms: 70 units of 2^-24 per step and six
    # steps, of values below max|X0|; bfloat16: a rounding may land on a
    # neighbouring value, at most 2^-7 |y| per sweep
    top = np.abs(X0).max()
    tol = 6 * 70 * 2.0**-24 * top if dtype == "f32" else 3 * 2.0**-7 * top
    assert np.abs(X.float().cpu().numpy() - ref).max() <= tol
