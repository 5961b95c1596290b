"""Which solver Alg. 1's solves take, and that both give the same: in one launch
up to 16,384 nodes where every workgroup's rows fit, by launches above and
where hub rows do not fit."""
import numpy as np
import pytest

import test_gpu_cg_resident as R
from workloads import graphs as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _graph(name):
    n, chords, hubs = R.CASES[name]
    u, v = R._case(n, chords, hubs, 4)
    rng = np.random.default_rng(5)
    w = rng.uniform(0.5, 2.0, u.size).astype(np.float32)
    return W.csr_from_edges(n, u, v, w), rng.uniform(0.5, 2.0, u.size)


def _scale(name):
    from paper_1812_08942_amd import graphreduce as G

    g, wP = _graph(name)
    dg = G.DeviceGraph.from_numpy(g.row_ptr, g.col, g.w, "cuda:0")
    edges = G.gr_edge_list(dg)

    def run():
        w = torch.from_numpy(wP.copy()).to("cuda:0")
        rep = G.gr_sgd_scale(dg, dg, edges, w, k_max=1, seed=9)
        return rep["lambda_n"][0], w.cpu().numpy()

    return run


@pytest.mark.parametrize("name", ["2", "64", "65", "1000_hubs", "4097", "16384"])
def test_both_ways_agree(name, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    run = _scale(name)
    out = {}
    for mode in (None, "1", "0"):
        print(f"[gpu-case] CG path {name} {mode}", flush=True)
        if mode:
            monkeypatch.setenv("GR_CG_RESIDENT", mode)
        out[mode] = run()
    # the default is the one launch, whose sums have a fixed order
    assert out[None][0] == out["1"][0]
    assert np.array_equal(out[None][1], out["1"][1])
    # lambda_n: as against the direct solves.  The weights change by at most
    # a tenth of their mean, in proportion to squared differences of the
    # solves, which are good to some 1e-10.
    assert abs(out["0"][0] - out["1"][0]) <= 1e-9 * out["0"][0]
    assert np.abs(out["0"][1] - out["1"][1]).max() <= 1e-8 * out["0"][1].max()


@pytest.mark.parametrize("name", ["16385", "16384_unfit"])
def test_by_launches_where_they_do_not_fit(name, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_08942_amd import graphreduce as G

    run = _scale(name)
    print(f"[gpu-case] CG path {name}", flush=True)
    want = run()
    monkeypatch.setenv("GR_CG_RESIDENT", "0")
    got = run()
    assert want[0] == got[0] and np.array_equal(want[1], got[1])
    monkeypatch.setenv("GR_CG_RESIDENT", "1")
    with pytest.raises(G.GraphReduceError) as e:
        run()
    assert e.value.code == -6


def test_a_wait_that_runs_out_goes_on_by_launches(monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_08942_amd import graphreduce as G

    g, wP = _graph("4097")
    dg = G.DeviceGraph.from_numpy(g.row_ptr, g.col, g.w, "cuda:0")
    edges = G.gr_edge_list(dg)
    out = {}
    for name, value in (("GR_CG_RESIDENT", "0"), ("GR_CG_SPIN_LIMIT", "1")):
        print(f"[gpu-case] CG wait {name}={value}", flush=True)
        with monkeypatch.context() as m:
            m.setenv(name, value)
            w = torch.from_numpy(wP.copy()).to("cuda:0")
            rep = G.gr_sgd_scale(dg, dg, edges, w, k_max=3, seed=9)
            keep, _, spars = G.gr_sparsify(dg, rounds=2, add_frac=0.05, seed=7)
            out[name] = rep, w.cpu().numpy(), keep.cpu().numpy(), spars
    a, b = out["GR_CG_RESIDENT"], out["GR_CG_SPIN_LIMIT"]
    assert a[0] == b[0] and a[3] == b[3]
    assert np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])
