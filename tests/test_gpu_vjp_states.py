"""The smoothing's backward with states rebuilt from kept ones gives the bits
of the backward with every state stored, whatever the number of sweeps (no
spare state free, one, two, several rebuilds from one)."""
import numpy as np
import pytest

from workloads import graphs as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sweeps", [0, 1, 2, 3, 4, 5, 8, 13])
@pytest.mark.parametrize("K,dtype", [(4, "f32"), (16, "f32"), (8, "bf16"), (32, "bf16")])
def test_rebuilt_states_are_the_stored_ones(sweeps, K, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_08942_amd import graphreduce as G

    g = W.with_isolated(W.chung_lu(1501, mean_deg=30.0, seed=8), 2)
    print(f"[gpu-case] rebuilt states S={sweeps} K={K} {dtype}", flush=True)
    dg = G.DeviceGraph.from_numpy(g.row_ptr, g.col, g.w, "cuda:0")
    edges = G.gr_edge_list(dg)
    colours, nc = G.gr_colour_greedy(dg, 3)
    X0 = G.gr_init_vectors(g.n, K, 5, dtype, "cuda:0")
    cot = torch.randn(g.n, K, generator=torch.Generator(device="cuda:0").manual_seed(1),
                      device="cuda:0")
    a = G.gr_smooth_vjp(dg, edges, colours, nc, X0, cot, sweeps, store_states=True)
    b = G.gr_smooth_vjp(dg, edges, colours, nc, X0, cot, sweeps, store_states=False)
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    if sweeps == 0:
        assert torch.equal(a[1], cot) and not a[0].any()
    else:
        assert np.isfinite(a[0].cpu().numpy()).all() and a[0].any()
