"""One colour step over rows of every degree from 1 to 140, against the exact
means: tight enough that a tail entry left out or counted twice shows in any
row, in bfloat16 too.  Launch by launch and in one launch."""
import numpy as np
import pytest

from oracle import oracle as O
from workloads import graphs as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("flow", ["0", "1"])
@pytest.mark.parametrize("K,dtype", [(4, "f32"), (16, "f32"), (64, "f32"), (8, "bf16"),
                                     (32, "bf16"), (64, "bf16")])
def test_one_step(K, dtype, flow, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_08942_amd import graphreduce as G

    m = 140
    u, v = np.nonzero(np.tril(np.ones((m, m))))  # left u has u + 1 entries, right v m - v
    w = np.random.default_rng(3).uniform(0.5, 2.0, u.size).astype(np.float32)
    g = W.csr_from_edges(2 * m, u, v + m, w)
    A = np.zeros((m, m))
    A[u, v] = w
    X0 = torch.from_numpy(O.init_vectors(g.n, K, 7).astype(np.float32)).to("cuda:0")
    if dtype == "bf16":
        X0 = X0.to(torch.bfloat16)
    x = X0.float().cpu().numpy().astype(np.float64)
    dg = G.DeviceGraph.from_numpy(g.row_ptr, g.col, g.w, "cuda:0")
    monkeypatch.setenv("GR_GS_FLOW", flow)
    for first in (0, 1):  # the side that goes first reads the start's values only
        print(f"[gpu-case] one step K={K} {dtype} flow={flow} side {first}", flush=True)
        colours = ((np.arange(2 * m) >= m) != (first == 1)).astype(np.int32)
        X = X0.clone()
        G.gr_smooth(dg, torch.from_numpy(colours).to("cuda:0"), 2, X, 1)
        got = X.float().cpu().numpy()[first * m:(first + 1) * m]
        B = A if first == 0 else A.T
        want = (B @ x[(1 - first) * m:(2 - first) * m]) / B.sum(1, keepdims=True)
        # float32 sums of vectors and weights, at most 140 terms each, and the
        # quotient; storing in bfloat16 moves a value by at most 2^-8 of it
        top = np.abs(x).max()
        tol = (2 * 140 + 2) * 2.0**-24 * top
        if dtype == "bf16":
            tol = tol + 2.0**-8 * np.abs(want)
        assert np.all(np.abs(got - want) <= tol)
        # an entry left out moves its row by more than that in some column
        last = np.array([np.nonzero(r)[0][-1] for r in B])
        move = (B[np.arange(m), last] / B.sum(1))[:, None] * (
            x[(1 - first) * m + last] - want)
        assert np.all((np.abs(move) > 4 * tol).any(1)[B.astype(bool).sum(1) > 1])
