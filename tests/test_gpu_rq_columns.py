"""Rayleigh quotients and their gradients for every kind of column count (one,
odd, even, a row per wave) and edge count (none, one, less and more than a
wave's, ragged), with U on and off a 16-byte boundary, against float64 sums
on the host."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m", [1, 2, 3, 10, 31, 63, 64])
@pytest.mark.parametrize("n,E", [(5, 0), (5, 1), (40, 63), (500, 4099), (70001, 200003)])
def test_columns_and_edges(m, n, E):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_08942_amd import graphreduce as G

    rng = np.random.default_rng(m + E)
    u = rng.integers(0, n - 1, E)
    v = u + 1 + rng.integers(0, 1 << 30, E) % (n - 1 - u)
    w = rng.uniform(0.5, 2.0, E)
    X = rng.standard_normal((n, m))
    dev = "cuda:0"
    edges = G.EdgeList(torch.from_numpy(u.astype(np.int32)).to(dev),
                       torch.from_numpy(v.astype(np.int32)).to(dev), None, n)
    wd, gR = torch.from_numpy(w).to(dev), torch.linspace(0.5, 2.0, m, dtype=torch.float64, device=dev)
    for offset in (0, 1):
        U = torch.zeros(n * m + 1, dtype=torch.float64, device=dev)[offset:offset + n * m].view(n, m)
        U.copy_(torch.from_numpy(X))
        for mode in (0, 1):
            print(f"[gpu-case] rq m={m} n={n} E={E} offset={offset} mode={mode}", flush=True)
            R, den = G.gr_rq_forward(edges, wd, U, mode)
            gw = G.gr_rq_backward(edges, U, R, den, gR, mode)
            d2, s2 = (X[u] - X[v]) ** 2, X[u] ** 2 + X[v] ** 2
            dr = (w[:, None] * s2).sum(0) if mode else (X * X).sum(0)
            safe = np.where(dr != 0, dr, 1.0)
            Rr = np.where(dr != 0, (w[:, None] * d2).sum(0) / safe, 0.0)
            t = d2 - (Rr * s2 if mode else 0.0)
            gr = (np.where(dr != 0, gR.cpu().numpy() / safe, 0.0) * t).sum(1)
            # at most 200,003 terms per sum, all of one sign: their relative
            # error stays below the number of terms in units of 2^-53
            tol = 200003 * 2.0**-53
            assert np.all(np.abs(den.cpu().numpy() - dr) <= tol * dr)
            assert np.all(np.abs(R.cpu().numpy() - Rr) <= 2 * tol * Rr)
            if E:
                scale = (np.where(dr != 0, gR.cpu().numpy() / safe, 0.0) * (d2 + Rr * s2)).sum(1)
                assert np.all(np.abs(gw.cpu().numpy() - gr) <= 4 * tol * scale)
