"""The Laplacian times a block of columns, through one Jacobi step, against
float64 sums on the host: every kind of column count (one, odd, even, a slot
per wave, more than half a wave) and rows without entries, short, at the
length from which a row takes a workgroup, and hubs."""
import numpy as np
import pytest

from workloads import graphs as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _graph():
    rng = np.random.default_rng(2)
    n = 3000
    u, v = [np.arange(n - 41)], [np.arange(1, n - 40)]  # a path; 40 nodes alone
    for hub, deg in ((5, 511), (700, 512), (1400, 513), (2900, 2500)):
        u.append(np.full(deg, hub))
        v.append(rng.choice(n - 40, deg, replace=False))
    u, v = np.concatenate(u), np.concatenate(v)
    key = np.unique(np.minimum(u, v) * n + np.maximum(u, v))
    key = key[key // n != key % n]
    w = rng.uniform(0.5, 2.0, key.size).astype(np.float32)
    return W.csr_from_edges(n, key // n, key % n, w)


@pytest.mark.parametrize("k", [1, 2, 3, 7, 18, 20, 33, 63, 64])
@pytest.mark.parametrize("offset", [0, 1])
def test_block_product(k, offset):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_08942_amd import graphreduce as G

    g = _graph()
    print(f"[gpu-case] block product k={k} offset={offset}", flush=True)
    dg = G.DeviceGraph.from_numpy(g.row_ptr, g.col, g.w, "cuda:0")
    X = np.random.default_rng(k).standard_normal((g.n, k))
    # offset 1: the array starts 8 bytes past a 16-byte boundary
    store = torch.zeros(g.n * k + 1, dtype=torch.float64, device="cuda:0")
    Y = store[offset:offset + g.n * k].view(g.n, k)
    Y.copy_(torch.from_numpy(X))
    G.gr_jacobi_filter(dg, Y, theta=0.5, iters=1)
    rows = np.repeat(np.arange(g.n), g.degrees())
    w = g.w.astype(np.float64)
    AX = np.zeros_like(X)
    np.add.at(AX, rows, w[:, None] * X[g.col])
    d = np.bincount(rows, weights=w, minlength=g.n)
    ref = np.where(d[:, None] > 0, X - 0.5 * (d[:, None] * X - AX) / np.where(d, d, 1)[:, None], X)
    # sums of at most 2,500 terms of weights up to 2 and values up to 5,
    # divided by the degree: a few units of 2^-53 per term
    assert np.abs(Y.cpu().numpy() - ref).max() <= 4 * 2500 * 2.0**-53 * np.abs(X).max()
