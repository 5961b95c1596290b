"""The solves of Alg. 1 that run in one launch, at the sizes where that
kernel's split can go wrong: fewer rows than workgroups, whole and ragged
rows per workgroup, its largest size and one more (by launches), rows of one
and of many pieces, and a graph whose hub rows do not fit one workgroup (by
launches too).  The reference solves the sparse systems directly (float64)."""
import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as spl

from oracle import oracle as O
from workloads import graphs as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _lap(n, u, v, w):
    A = sp.coo_matrix((np.r_[w, w], (np.r_[u, v], np.r_[v, u])), shape=(n, n)).tocsr()
    return (sp.diags(np.asarray(A.sum(1)).ravel()) - A).tocsc()


def _case(n, chords, hubs, seed):
    """(u, v) of a ring with chords of up to 40 steps (so that the reference
    factors with little fill) and hubs joined to every node."""
    rng = np.random.default_rng(seed)
    i = np.arange(n)
    c = rng.integers(0, n, chords)
    u = [i, c]
    v = [(i + 1) % n, (c + rng.integers(1, 41, chords)) % n]
    for h in hubs:
        u.append(np.full(n, h))
        v.append(i)
    u, v = np.concatenate(u), np.concatenate(v)
    key = np.unique(np.minimum(u, v) * n + np.maximum(u, v))
    key = key[key // n != key % n]
    return key // n, key % n


CASES = {
    "2": (2, 0, []), "63": (63, 100, []), "64": (64, 0, [5]), "65": (65, 200, []),
    "1000_hubs": (1000, 3000, [0, 64, 999]), "4097": (4097, 20000, [17]),
    "16384": (16384, 100000, [3]), "16385": (16385, 40000, [8]),
    "16384_unfit": (16384, 0, [0, 64, 128, 192, 256]),
}


@pytest.mark.parametrize("name", CASES)
def test_power_vector_of_one_launch_solves(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_08942_amd import graphreduce as G

    n, chords, hubs = CASES[name]
    u, v = _case(n, chords, hubs, 4)
    rng = np.random.default_rng(5)
    wG = rng.uniform(0.5, 2.0, u.size).astype(np.float32)
    wP = rng.uniform(0.5, 2.0, u.size)
    g = W.csr_from_edges(n, u, v, wG)
    print(f"[gpu-case] resident solves {name}: n={n} nnz={g.nnz}", flush=True)
    dg = G.DeviceGraph.from_numpy(g.row_ptr, g.col, g.w, "cuda:0")
    edges = G.gr_edge_list(dg)
    w = torch.from_numpy(wP.copy()).to("cuda:0")
    rep = G.gr_sgd_scale(dg, dg, edges, w, k_max=1, seed=9)
    LG, LP = _lap(n, u, v, wG.astype(np.float64)), _lap(n, u, v, wP)
    solve = spl.splu(LP[1:, 1:]).solve
    h = O.init_vectors(n, 1, 9)[:, 0]
    for _ in range(2):
        b = LG @ (h - h.mean())
        h = np.r_[0.0, solve((b - b.mean())[1:])]
    h -= h.mean()
    lam = (h @ (LG @ h)) / (h @ (LP @ h))
    # the solves stop at a relative residual of 1e-13; the preconditioned
    # systems have condition numbers of at most some hundreds (short rings,
    # or a hub two steps from everything)
    assert abs(rep["lambda_n"][0] - lam) <= 1e-9 * lam
    assert np.all(w.cpu().numpy() >= wP)
