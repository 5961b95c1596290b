"""Data restriction by two columns per load: column counts that allow it and
those that don't, arrays that are not aligned for it, aggregates of one piece
(finished where they are summed), of exactly 256, 257 and of thousands of
members.  The float64 sum in node order, over the member count and rounded
once, bit for bit up to 256 members; beyond, one rounding of the pieces' sum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d", [1, 2, 5, 6, 8, 784])
@pytest.mark.parametrize("shift", [0, 1])
def test_columns(d, shift):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_08942_amd import graphreduce as G

    sizes = [1, 2, 3, 4, 5, 255, 256, 257, 512, 513, 3000]
    rng = np.random.default_rng(d)
    agg = rng.permutation(np.repeat(np.arange(len(sizes)), sizes))
    n, nc = agg.size, len(sizes)
    F = rng.standard_normal((n, d)).astype(np.float32)
    flat = torch.empty(n * d + shift, dtype=torch.float32, device="cuda:0")
    Fd = flat[shift:].view(n, d)
    Fd.copy_(torch.from_numpy(F))
    print(f"[gpu-case] restriction d={d} shift={shift}", flush=True)
    out = G.gr_restrict_mean(torch.from_numpy(agg.astype(np.int32)).to("cuda:0"), nc,
                             Fd).cpu().numpy()
    s = np.zeros((nc, d))
    np.add.at(s, agg, F.astype(np.float64))
    ref = (s / np.array(sizes)[:, None]).astype(np.float32)
    small = np.array(sizes) <= 256
    assert np.array_equal(out[small], ref[small])
    assert np.all(np.abs(out - ref) <= np.spacing(np.abs(ref)) + 1e-12 * np.abs(F).max())
