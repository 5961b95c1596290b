"""The stable sort and the scans at the sizes where their form changes (one
workgroup with 2, 4 or 8 keys per thread, launches, one-workgroup and
two-launch scans), through the data restriction: members in node order give
the float64 sum in node order, bit for bit up to 256 members."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1, 63, 2048, 2049, 4096, 4097, 8192, 8193, 16385, 131072, 131073,
                               1500001])
def test_members_in_node_order(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_08942_amd import graphreduce as G

    rng = np.random.default_rng(n)
    F = rng.standard_normal((n, 3)).astype(np.float32)
    for nc in sorted({1, min(n, 2), min(n, 200), (n + 2) // 3, n}):
        agg = rng.integers(0, nc, n)
        agg[rng.permutation(n)[:nc]] = np.arange(nc)  # each has a member
        print(f"[gpu-case] restriction n={n} nc={nc}", flush=True)
        out = G.gr_restrict_mean(torch.from_numpy(agg.astype(np.int32)).to("cuda:0"), nc,
                                 torch.from_numpy(F).to("cuda:0")).cpu().numpy()
        s = np.zeros((nc, 3))
        np.add.at(s, agg, F.astype(np.float64))
        cnt = np.bincount(agg, minlength=nc)
        ref = (s / cnt[:, None]).astype(np.float32)
        small = cnt <= 256
        assert np.array_equal(out[small], ref[small])
        assert np.all(np.abs(out - ref) <= np.spacing(np.abs(ref)) + 1e-12 * np.abs(F).max())
