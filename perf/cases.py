"""The calls that programs make of this framework, as cases to be timed.

`listed()` gives the named cases, `draw(rng)` one more of the same ranges,
`prepare` what a program has in hand before the call (graph, colouring, edge
list, test vectors, weights: on the GPU, made from the seed alone), `run` one
pass through the public entry points, `work` the bytes and operations that a
pass cannot do without, `exact` the same results in float64 from plain torch.

Kinds
  reduce    gr_reduce: the whole node reduction of a graph.  The main call.
  smooth    autograd.smoothed_vectors, forward and backward: Gauss-Seidel
            smoothing of test vectors, gradients for edge weights and vectors.
  rq        autograd.rayleigh_quotients, forward and backward.
  eigs      gr_laplacian_eigs: the first nontrivial eigenvalues of a reduced
            graph, the measure of a reduction's quality.
  scale     gr_sgd_scale: the edge scaling of a sparsifier of a reduced graph.
  flow      gr_spectral_reduce: reduction, sparsification and scaling in one.
  restrict  gr_restrict_mean: data points averaged over the aggregates.

Graphs: 2-D and 3-D meshes, k-nearest-neighbour graphs of points in the plane
and of image-shaped data, power-law graphs; K, sweeps, ratio and storage type
as the workloads of workloads/graphs.py set them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1812_08942_amd import autograd as A
from paper_1812_08942_amd import graphreduce as G

DEV = "cuda:0"


# ------------------------------------------------------------------- cases

def listed():
    return [
        # the smallest reduction: a 64 x 64 finite-element mesh with its
        # checkerboard colouring; launches and host round trips count
        {"name": "reduce_mesh2d_64", "kind": "reduce", "graph": "grid2d", "nx": 64, "ny": 64,
         "K": 8, "dtype": "f32", "ratio": 4.0},
        # an ordinary one: nearest-neighbour graph of points in the plane,
        # greedy colouring, three levels of small kernels
        {"name": "reduce_knn_200k", "kind": "reduce", "graph": "knn", "n": 200000,
         "K": 16, "dtype": "f32", "ratio": 32.0},
        # MNIST-shaped data, 70k points in 784 dimensions: hubs, many colours
        {"name": "reduce_images_70k", "kind": "reduce", "graph": "images", "n": 70000,
         "K": 16, "dtype": "f32", "ratio": 16.0},
        # a citation or social network: power law, dense second level
        {"name": "reduce_powerlaw_434k", "kind": "reduce", "graph": "powerlaw", "n": 434000,
         "mean_deg": 73.7, "K": 16, "dtype": "f32", "ratio": 33.385},
        # the largest: a 256^3 mesh, bfloat16 vectors, prescribed colouring
        {"name": "reduce_mesh3d_256", "kind": "reduce", "graph": "grid3d", "nx": 256, "ny": 256,
         "nz": 256, "K": 32, "dtype": "bf16", "ratio": 170.0},
        # learning edge weights through the smoothing, power-law graph,
        # states recomputed in the backward pass
        {"name": "smooth_grad_powerlaw_434k", "kind": "smooth", "graph": "powerlaw", "n": 434000,
         "mean_deg": 73.7, "K": 16, "dtype": "f32", "store": False},
        # the same on a 3-D mesh of odd sides, bfloat16 states that are kept
        {"name": "smooth_grad_mesh3d_127", "kind": "smooth", "graph": "grid3d", "nx": 127,
         "ny": 129, "nz": 125, "K": 32, "dtype": "bf16", "store": True},
        # spectral quality of edge weights on a reduced graph: the inner call
        # of a training loop, tens of microseconds
        {"name": "rq_grad_13k", "kind": "rq", "n": 13000, "mean_deg": 197.0, "m": 10, "mode": 0},
        # the quality report of a reduced power-law graph
        {"name": "eigs_13k", "kind": "eigs", "n": 13000, "mean_deg": 197.0, "n_eig": 10},
        # Alg. 1 on the spanning sparsifier of the same
        {"name": "scale_13k", "kind": "scale", "n": 13000, "mean_deg": 197.0, "extra": 0.1},
        # Alg. 2 on the image graph: reduce, sparsify, scale
        {"name": "flow_images_70k", "kind": "flow", "graph": "images", "n": 70000,
         "K": 16, "dtype": "f32", "ratio": 16.0},
        # the reduced data set that goes to the visualisation (Alg. 6)
        {"name": "restrict_images_70k", "kind": "restrict", "n": 70000, "d": 784, "nc": 4375},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, names, most=1.0):
    g = rng.choice(names)
    if g == "grid2d":
        return {"graph": g, "nx": _log(rng, 40, 1500 * most), "ny": _log(rng, 40, 1500 * most)}
    if g == "grid3d":
        s = lambda: _log(rng, 16, 256 * most)  # noqa: E731
        return {"graph": g, "nx": s(), "ny": s(), "nz": s()}
    if g == "knn":
        return {"graph": g, "n": _log(rng, 2000, 400000 * most)}
    if g == "images":
        return {"graph": g, "n": _log(rng, 3000, 70000)}
    return {"graph": "powerlaw", "n": _log(rng, 5000, 434000 * most),
            "mean_deg": round(rng.uniform(20.0, 73.7), 1)}


def _draw_vectors(rng):
    dt = rng.choice(["f32", "f32", "bf16"])
    return {"K": rng.choice([8, 16, 32, 64] if dt == "bf16" else [4, 8, 16, 32]), "dtype": dt}


def draw(rng):
    kind = rng.choice(["reduce"] * 6 + ["smooth"] * 2 + ["rq", "eigs", "scale", "flow", "restrict"])
    if kind == "reduce":
        return {"kind": kind, **_draw_graph(rng, ["grid2d", "grid3d", "knn", "images", "powerlaw"]),
                **_draw_vectors(rng), "ratio": round(rng.uniform(4.0, 64.0), 2)}
    if kind == "smooth":
        return {"kind": kind, **_draw_graph(rng, ["grid3d", "knn", "powerlaw"], 0.5),
                **_draw_vectors(rng), "store": rng.random() < 0.5}
    if kind == "rq":
        return {"kind": kind, "n": _log(rng, 1000, 100000), "mean_deg": round(rng.uniform(8, 200), 1),
                "m": rng.randint(2, 32), "mode": rng.randint(0, 1)}
    if kind == "eigs":
        return {"kind": kind, "n": _log(rng, 1000, 13000), "mean_deg": round(rng.uniform(60, 200), 1),
                "n_eig": rng.randint(5, 10)}
    if kind == "scale":
        return {"kind": kind, "n": _log(rng, 1000, 13000), "mean_deg": round(rng.uniform(60, 200), 1),
                "extra": round(rng.uniform(0.05, 0.2), 3)}
    if kind == "flow":
        return {"kind": kind, "graph": "images", "n": _log(rng, 4000, 70000), "K": 16,
                "dtype": "f32", "ratio": round(rng.uniform(8.0, 20.0), 2)}
    n = _log(rng, 5000, 434000)
    return {"kind": kind, "n": n, "d": _log(rng, 2, 200), "nc": max(2, int(n / rng.uniform(4, 64)))}


# ------------------------------------------------------------------ graphs

def _gen(seed, sub):
    return torch.Generator(device=DEV).manual_seed(1000003 * int(seed) + sub)


def _csr(n, lo, hi, w):
    """DeviceGraph of the undirected edges (lo, hi), each pair once."""
    rows, cols = torch.cat([lo, hi]), torch.cat([hi, lo])
    key, order = torch.sort(rows * n + cols)
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(rows, minlength=n), 0, out=rp[1:])
    return G.DeviceGraph(rp.to(torch.int32), (key % n).to(torch.int32),
                         torch.cat([w, w])[order].to(torch.float32).contiguous())


def _edges_of(case):
    """Undirected edges of the case's graph: a number of the case alone, so
    that the arrays of every seed have one size."""
    kind = case.get("graph", "powerlaw")
    if kind in ("grid2d", "grid3d"):
        d = [case["nx"], case["ny"], case.get("nz", 1)]
        n = d[0] * d[1] * d[2]
        return sum(n - n // k for k in d)
    n = case["n"]
    per = {"knn": 5.3, "images": 8.4}.get(kind) or min(case["mean_deg"], n / 8) / 2
    return int(n * per)


def _some(m, want, gen):
    """`want` of the numbers 0 .. m-1, ascending."""
    if m < want:
        raise ValueError("%d edges, fewer than %d" % (m, want))
    return torch.sort(torch.randperm(m, generator=gen, device=DEV)[:want]).values


def _knn_weights(n, nbr, dist2, edges, gen):
    """The union-symmetrised neighbour graph, w = exp(-d^2 / sigma^2), with
    `edges` of its edges."""
    k = nbr.shape[1]
    i = torch.arange(n, device=DEV).repeat_interleave(k)
    j = nbr.reshape(-1)
    sigma = dist2.double().sqrt().mean()
    key, inv = torch.unique(torch.minimum(i, j) * n + torch.maximum(i, j), return_inverse=True)
    d2 = torch.zeros(key.numel(), dtype=torch.float64, device=DEV)
    d2[inv] = dist2.double().reshape(-1)  # d(i,j) and d(j,i) are the same bits
    at = _some(key.numel(), edges, gen)
    key, d2 = key[at], d2[at]
    return _csr(n, key // n, key % n, torch.exp(-d2 / sigma**2).clamp_min(1e-37))


def knn_graph(n, edges, seed, k=10):
    """Points spread evenly over the plane, one in each cell of a square
    lattice, in random order; the k nearest of the 7 x 7 cells around."""
    g = _gen(seed, 1)
    nx = int(math.isqrt(n - 1)) + 1
    cell = torch.arange(n, device=DEV)
    cx, cy = cell % nx, cell // nx
    p = torch.rand(n, 2, generator=g, device=DEV, dtype=torch.float64)
    p += torch.stack([cx, cy], 1)
    off = torch.tensor([(x, y) for y in range(-3, 4) for x in range(-3, 4) if x or y], device=DEV)
    qx, qy = cx[:, None] + off[:, 0], cy[:, None] + off[:, 1]
    q = qx + nx * qy
    ok = (qx >= 0) & (qx < nx) & (qy >= 0) & (q < n)
    q = torch.where(ok, q, 0)
    d2 = ((p[:, None, :] - p[q]) ** 2).sum(2).masked_fill(~ok, float("inf"))
    d2, at = torch.sort(d2, 1)
    name = torch.randperm(n, generator=g, device=DEV)
    nbr = torch.empty(n, k, dtype=torch.int64, device=DEV)
    nbr[name] = name[q.gather(1, at[:, :k])]
    dist2 = torch.empty(n, k, dtype=torch.float64, device=DEV)
    dist2[name] = d2[:, :k]
    return _knn_weights(n, nbr, dist2, edges, g)


def images_graph(n, edges, seed, k=10, dim=784):
    """k nearest neighbours of a 10-component Gaussian mixture in 784
    dimensions whose coordinates are whole numbers, as pixels are, so that
    the distances are exact in float32."""
    g = _gen(seed, 2)
    means = 0.12 * torch.randn(10, dim, generator=g, device=DEV)
    pts = means[torch.arange(n, device=DEV) % 10] + torch.randn(n, dim, generator=g, device=DEV)
    pts = torch.round(16.0 * pts)
    sq = (pts * pts).sum(1)
    nbr = torch.empty(n, k, dtype=torch.int64, device=DEV)
    dist2 = torch.empty(n, k, dtype=torch.float64, device=DEV)
    ids = torch.arange(n, device=DEV)
    for s in range(0, n, 4096):
        e = min(n, s + 4096)
        d2 = sq[s:e, None] + sq[None, :] - 2.0 * (pts[s:e] @ pts.T)
        d2[ids[s:e] - s, ids[s:e]] = 1e9
        key = d2.double() * n + ids  # ties by number
        best = torch.topk(key, k, dim=1, largest=False).values
        dist2[s:e] = torch.floor(best / n)
        nbr[s:e] = (best - dist2[s:e] * n).long()
    return _knn_weights(n, nbr, dist2, edges, g)


def powerlaw_graph(n, edges, seed, beta=2.5):
    """Chung-Lu graph: expected degrees with a power-law tail of exponent
    beta, largest sqrt(2 edges), weights U[0.5, 2]."""
    ex, mean, top = 1.0 / (beta - 1.0), 2.0 * edges / n, math.sqrt(2.0 * edges)
    i = torch.arange(n, dtype=torch.float64, device=DEV)
    lo, hi = 1e-3, 1e9
    for _ in range(60):
        mid = math.sqrt(lo * hi)
        if float((top * ((i + mid) / mid) ** -ex).mean()) < mean:
            lo = mid
        else:
            hi = mid
    theta = (top * ((i + lo) / lo) ** -ex).cpu().numpy()
    cdf = torch.from_numpy(np.cumsum(theta) / theta.sum()).to(DEV)
    g = _gen(seed, 3)
    ends = torch.searchsorted(cdf, torch.rand(2, int(1.3 * edges), generator=g, device=DEV,
                                              dtype=torch.float64), right=True).clamp_max(n - 1)
    key = torch.unique(torch.minimum(ends[0], ends[1]) * n + torch.maximum(ends[0], ends[1]))
    key = key[key // n != key % n]
    key = key[_some(key.numel(), edges, g)]
    w = 0.5 + 1.5 * torch.rand(edges, generator=g, device=DEV)
    return _csr(n, key // n, key % n, w)


# rank of the parity triple 4 (x&1) + 2 (y&1) + (z&1) in the reflected Gray
# sequence: consecutive colours differ in one parity
GRAY = (0, 1, 3, 2, 7, 6, 4, 5)


def grid_graph(nx, ny, nz, seed, weights):
    """Mesh of nx x ny x nz nodes, v = x + nx (y + ny z), unit or lognormal
    weights, with its parity colouring: (graph, colours, number)."""
    g = _gen(seed, 4)
    N = nx * ny * nz
    ids = torch.arange(N, dtype=torch.int32, device=DEV).reshape(nz, ny, nx)
    col = torch.full((nz, ny, nx, 6), -1, dtype=torch.int32, device=DEV)
    w = torch.zeros((nz, ny, nx, 6), device=DEV)
    for axis, down, up in ((0, 0, 5), (1, 1, 4), (2, 2, 3)):
        m = ids.shape[axis] - 1
        if m < 1:
            continue
        a, b = ids.narrow(axis, 0, m), ids.narrow(axis, 1, m)
        we = (torch.exp(torch.randn(a.shape, generator=g, device=DEV)) if weights == "lognormal"
              else torch.ones(a.shape, device=DEV))
        col.narrow(axis, 1, m)[..., down] = a
        w.narrow(axis, 1, m)[..., down] = we
        col.narrow(axis, 0, m)[..., up] = b
        w.narrow(axis, 0, m)[..., up] = we
    ok = (col >= 0).reshape(N, 6)
    rp = torch.zeros(N + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(ok.sum(1), 0, out=rp[1:])
    graph = G.DeviceGraph(rp.to(torch.int32), col.reshape(N, 6)[ok].contiguous(),
                          w.reshape(N, 6)[ok].contiguous())
    v = torch.arange(N, device=DEV)
    x, y, z = v % nx, v // nx % ny, v // (nx * ny)
    if nz == 1:
        return graph, ((x + y) % 2).to(torch.int32), 2
    rank = torch.tensor(GRAY, dtype=torch.int32, device=DEV)
    return graph, rank[4 * (x & 1) + 2 * (y & 1) + (z & 1)], 8


def make_graph(case, seed):
    """(graph, prescribed colours or None, their number)."""
    kind = case.get("graph", "powerlaw")
    if kind == "grid2d":
        # unit weights, as a finite-difference mesh has them: only the test
        # vectors come from the seed
        return grid_graph(case["nx"], case["ny"], 1, seed, "unit")
    if kind == "grid3d":
        return grid_graph(case["nx"], case["ny"], case["nz"], seed, "lognormal")
    if kind == "knn":
        return knn_graph(case["n"], _edges_of(case), seed), None, 0
    if kind == "images":
        return images_graph(case["n"], _edges_of(case), seed), None, 0
    return powerlaw_graph(case["n"], _edges_of(case), seed), None, 0


def _edge_values(edges, w):
    """float64 per undirected edge from the entries' weights."""
    wE = torch.empty(edges.E, dtype=torch.float64, device=DEV)
    wE[edges.edge_of_entry.long()] = w.double()
    return wE


# ----------------------------------------------------------------- a pass

SWEEPS = 5


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "seed": int(seed)}
    if kind == "restrict":
        n, nc, d = case["n"], case["nc"], case["d"]
        g = _gen(seed, 5)
        # aggregate sizes spread as a reduction leaves them: each has a
        # member, some have many
        u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
        agg = (nc * u**2).long().clamp_max(nc - 1)
        agg[:nc] = torch.arange(nc, device=DEV)
        s["agg"] = agg[torch.randperm(n, generator=g, device=DEV)].to(torch.int32)
        s["F"] = torch.randn(n, d, generator=g, device=DEV)
        return s
    s["g"], s["colours"], s["nc"] = make_graph(case, seed)
    g = s["g"]
    if kind == "reduce":
        # the output buffers that a program reducing graph after graph keeps
        s["out"] = (torch.zeros(g.n, dtype=torch.int32, device=DEV),
                    torch.zeros(g.n + 1, dtype=torch.int32, device=DEV),
                    torch.zeros(g.nnz, dtype=torch.int32, device=DEV),
                    torch.zeros(g.nnz, device=DEV))
    elif kind == "smooth":
        if s["colours"] is None:
            s["colours"], s["nc"] = G.gr_colour_greedy(g, seed, case["graph"] == "powerlaw")
        s["edges"] = G.gr_edge_list(g)
        s["w"] = _edge_values(s["edges"], g.w).to(torch.float32)
        s["X0"] = G.gr_init_vectors(g.n, case["K"], seed, case["dtype"], DEV)
        gen = _gen(seed, 6)
        s["cot"] = torch.randn(g.n, case["K"], generator=gen, device=DEV).to(s["X0"].dtype)
    elif kind == "rq":
        s["edges"] = G.gr_edge_list(g)
        s["w"] = _edge_values(s["edges"], g.w)
        gen = _gen(seed, 7)
        s["U"] = torch.randn(g.n, case["m"], generator=gen, device=DEV, dtype=torch.float64)
        s["cot"] = torch.rand(case["m"], generator=gen, device=DEV, dtype=torch.float64) + 0.5
    elif kind == "scale":
        e = G.gr_edge_list(g)
        wE = _edge_values(e, g.w)
        keep, _ = G.gr_spanning_forest(g)
        rest = torch.where(keep.bool(), -1.0, wE)
        more = torch.sort(rest, descending=True, stable=True).indices
        keep = keep.clone()
        keep[more[:int(round(case["extra"] * int((rest > 0).sum())))]] = 1
        s["P"], s["edges"] = G.gr_subgraph(g, keep)
        s["w"] = wE[keep.bool()]
    return s


def _padded(values, size=21):
    """One entry per iteration, of at most 20, and the last one's."""
    return np.array(values + [0.0] * (size - len(values)))


def run(s):
    case, kind, seed = s["case"], s["case"]["kind"], s["seed"]
    if kind == "reduce":
        r = G.gr_reduce(s["g"], case["K"], SWEEPS, case["ratio"], seed + 10, seed + 20,
                        dtype=case["dtype"], colours=s["colours"], n_colours=s["nc"],
                        largest_degree_first=case["graph"] == "powerlaw", out=s["out"])
        return (r.coarse.n, r.coarse.nnz, *s["out"])
    if kind == "smooth":
        w = s["w"].detach().requires_grad_()
        X0 = s["X0"].detach().requires_grad_()
        X = A.smoothed_vectors(w, X0, s["g"], s["edges"], s["colours"], s["nc"], SWEEPS,
                               case["store"])
        return (X.detach(), *torch.autograd.grad(X, (w, X0), s["cot"]))
    if kind == "rq":
        w = s["w"].detach().requires_grad_()
        R = A.rayleigh_quotients(w, s["U"], s["edges"], case["mode"])
        return (R.detach(), *torch.autograd.grad(R, (w,), s["cot"]))
    if kind == "eigs":
        return G.gr_laplacian_eigs(s["g"], case["n_eig"], seed=seed + 1)[0]
    if kind == "scale":
        w = s["w"].clone()
        rep = G.gr_sgd_scale(s["g"], s["P"], s["edges"], w, seed=seed + 1)
        return w, _padded(rep["lambda_n"]), _padded(rep["lambda_1"])
    if kind == "flow":
        r = G.gr_spectral_reduce(s["g"], case["K"], SWEEPS, case["ratio"], seed + 10, seed + 20,
                                 dtype=case["dtype"])
        pad, n = torch.nn.functional.pad, case["n"]
        return (r.S.n, r.S.nnz, r.agg, pad(r.S.row_ptr, (0, n - r.S.n)),
                pad(r.S.col, (0, 2 * n - r.S.nnz)), pad(r.S.w, (0, 2 * n - r.S.nnz)))
    return G.gr_restrict_mean(s["agg"], case["nc"], s["F"])


# ------------------------------------------------------- necessary work

def work(case):
    kind = case["kind"]
    if kind == "restrict":
        n, nc, d = case["n"], case["nc"], case["d"]
        return {"bytes": 4.0 * (n * d + nc * d + n), "flops": float(n * d + nc * d)}
    n = case["n"] if "n" in case else case["nx"] * case["ny"] * case.get("nz", 1)
    nnz = 2 * _edges_of(case)
    graph = 4.0 * (n + 1) + 8.0 * nnz
    if kind in ("reduce", "flow"):
        # the graph in, the map and the reduced graph out; the first
        # level's smoothing and affinities
        return {"bytes": graph + 4.0 * n + graph / case["ratio"],
                "flops": float(nnz * case["K"] * (2 * SWEEPS + 4))}
    E = nnz / 2
    if kind == "smooth":
        v = n * case["K"]
        return {"bytes": graph + 4.0 * nnz + 4.0 * n + 8.0 * E
                + 4.0 * v * (2 if case["dtype"] == "bf16" else 4),
                "flops": float(nnz * case["K"] * 6 * SWEEPS)}
    if kind == "rq":
        return {"bytes": 8.0 * n * case["m"] + E * (8 + 16), "flops": 8.0 * E * case["m"]}
    if kind == "eigs":
        # one block product at least
        return {"bytes": graph, "flops": 2.0 * nnz * case["n_eig"]}
    # every iteration needs the products and solves of its power vector
    p_edges = n + case["extra"] * E
    return {"bytes": graph + 32.0 * p_edges, "flops": 20.0 * 2 * (2 * nnz + 4 * p_edges)}


# ------------------------------------------------------ results in 64 bits

def exact(case, seed):
    kind = case["kind"]
    if kind in ("reduce", "flow"):
        # maps and structures are whole numbers; the reduced weights have no
        # value of their own apart from the map
        return None
    if kind == "eigs":
        return _exact_eigs(case, seed)
    if kind == "scale":
        return _exact_scale(case, seed) if case["n"] <= 6000 else None
    s = prepare(case, seed)
    if kind == "restrict":
        at = s["agg"].long()
        out = torch.zeros(case["nc"], case["d"], dtype=torch.float64, device=DEV)
        out.index_add_(0, at, s["F"].double())
        return out / torch.bincount(at, minlength=case["nc"])[:, None]
    if kind == "rq":
        eu, ev, U = s["edges"].eu.long(), s["edges"].ev.long(), s["U"]
        w = s["w"].clone().requires_grad_()
        num = (w[:, None] * (U[eu] - U[ev]) ** 2).sum(0)
        den = ((w[:, None] * (U[eu] ** 2 + U[ev] ** 2)).sum(0) if case["mode"]
               else (U * U).sum(0))
        R = num / den
        return (R.detach(), *torch.autograd.grad(R, (w,), s["cot"]))
    return _exact_smooth(s)


def _exact_smooth(s):
    """Gauss-Seidel by colours and its gradients, float64 throughout.  Per
    colour step: x_c = D_c^-1 A_c x on the step's rows."""
    g, c = s["g"], s["colours"].long()
    n = g.n
    deg = (g.row_ptr[1:] - g.row_ptr[:-1]).long()
    row = torch.repeat_interleave(torch.arange(n, device=DEV), deg)
    col, eoe = g.col.long(), s["edges"].edge_of_entry.long()
    wE = s["w"].double()
    dsum = torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, row, wE[eoe])
    X = s["X0"].double()
    order = torch.argsort(c[row], stable=True)
    cut = torch.cumsum(torch.bincount(c[row], minlength=s["nc"]), 0).tolist()
    steps = []
    for k in range(s["nc"]):
        e = order[(cut[k - 1] if k else 0):cut[k]]
        rows = torch.nonzero((c == k) & (deg > 0)).reshape(-1)
        at = torch.empty(n, dtype=torch.int64, device=DEV)
        at[rows] = torch.arange(rows.numel(), device=DEV)
        steps.append((rows, at[row[e]], col[e], eoe[e], dsum[rows]))
    kept = []
    for _ in range(SWEEPS):
        for rows, loc, j, ee, d in steps:
            new = torch.zeros(rows.numel(), X.shape[1], dtype=torch.float64, device=DEV)
            new.index_add_(0, loc, wE[ee][:, None] * X[j])
            new /= d[:, None]
            kept.append(X[rows])
            X[rows] = new
    out = X.clone()
    # undo the steps: adjoint H of the state, gradient of every edge weight
    H = s["cot"].double()
    gw = torch.zeros_like(wE)
    for i in range(SWEEPS * len(steps) - 1, -1, -1):
        rows, loc, j, ee, d = steps[i % len(steps)]
        h = H[rows] / d[:, None]
        new = X[rows]
        X[rows] = kept[i]
        gw.index_add_(0, ee, (h[loc] * (X[j] - new[loc])).sum(1))
        H[rows] = 0.0
        H.index_add_(0, j, wE[ee][:, None] * h[loc])
    return out, gw, H


def _dense(n, rows, cols, w):
    """Laplacian of the entries as a dense float64 matrix."""
    L = torch.zeros(n, n, dtype=torch.float64, device=DEV)
    L[rows, cols] = -w
    L.diagonal().copy_(torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, rows, w))
    return L


def _rows(g):
    return torch.repeat_interleave(torch.arange(g.n, device=DEV),
                                   (g.row_ptr[1:] - g.row_ptr[:-1]).long())


def _exact_eigs(case, seed):
    """Inverse iteration with a block, on the complement of the constant (a
    graph with parts that hang together by nothing has no value here)."""
    g = make_graph(case, seed)[0]
    n, m = g.n, min(80, g.n // 4)
    if int((g.row_ptr[1:] == g.row_ptr[:-1]).sum()):
        return None
    L = _dense(n, _rows(g), g.col.long(), g.w.double())
    C = torch.linalg.cholesky(L + L.diagonal().mean() / n)
    X = torch.randn(n, m, generator=_gen(seed, 8), device=DEV, dtype=torch.float64)
    for _ in range(120):
        X = torch.cholesky_solve(X - X.mean(0), C)
        X = torch.linalg.qr(X - X.mean(0)).Q
    H = (X.T @ (L @ X)).cpu().numpy()
    return np.linalg.eigvalsh(0.5 * (H + H.T))[:case["n_eig"]]


def _splitmix(seed, n):
    """Outputs 0 .. n-1 of SplitMix64."""
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + np.arange(1, n + 1, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


def _exact_scale(case, seed):
    """Alg. 1 with the defaults of gr_sgd_scale and dense solves."""
    s = prepare(case, seed)
    g, eu, ev = s["g"], s["edges"].eu.long(), s["edges"].ev.long()
    n, w = g.n, s["w"].clone()
    both, other = torch.cat([eu, ev]), torch.cat([ev, eu])
    LG = _dense(n, _rows(g), g.col.long(), g.w.double())
    dG = LG.diagonal()
    if float(dG.min()) <= 0.0:
        return None
    m = (_splitmix(seed + 1, n) >> np.uint64(40)).astype(np.float64)
    h0 = torch.from_numpy((2 * m + 1 - 2.0**24) / 2.0**24).to(DEV)
    h0 = h0 - h0.mean()
    sums = lambda v: torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(  # noqa: E731
        0, both, torch.cat([v, v]))
    delta = 0.5 ** (1.0 / 20)
    dP = sums(w)
    lam1 = float((dG / dP).min())
    lam_n, lam_1, dw, top = [], [lam1], torch.zeros_like(w), None
    for _ in range(20):
        LP = _dense(n, both, other, torch.cat([w, w]))
        C = torch.linalg.cholesky(LP + LP.diagonal().mean() / n)
        h = h0
        for _ in range(2):
            h = torch.cholesky_solve((LG @ h)[:, None], C)[:, 0]
            h = h - h.mean()
        h = h / torch.sqrt(h @ (LP @ h))
        lam = float(h @ (LG @ h))
        stop = bool(lam_n) and (lam_n[-1] - lam) / lam < 1e-3
        lam_n.append(lam)
        if stop:
            break
        sens = -lam * (h[eu] - h[ev]) ** 2
        if top is None:
            top = eta = 0.1 * float(w.mean()) / float(sens.abs().max())
        dw = 0.9 * dw - eta * sens
        ask = dw.clamp_min(0.0)
        S, cap = sums(ask), dG / (lam1 * delta) - dP
        fac = torch.where(S > 0, cap / torch.where(S > 0, S, 1.0), float("inf"))
        lim = torch.where(ask > 0, torch.minimum(fac[eu], fac[ev]) * ask, 0.0)
        dw = torch.minimum(dw, lim).clamp_min(0.0)
        w = w + dw
        dP = dP + sums(dw)
        eta = lam / lam_n[0] * top
        lam1 = float((dG / dP).min())
        lam_1.append(lam1)
    return w, _padded(lam_n), _padded(lam_1)
