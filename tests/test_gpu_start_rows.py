"""Start centroids at the edges of the inference split (one histogram per
block below 512, four per block from there on, with a ragged last block):
bitwise the network's own outputs followed by the post-processing in FP32,
with histograms that leave no valid start among them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _post(y, h, C):
    """Sorted 255 y, clamped to the levels present, gaps >= 1; NaN where that cannot be."""
    f = np.float32
    at = np.flatnonzero(h > 0)
    lo, hi = (f(at[0]), f(at[-1])) if at.size else (f(255), f(0))
    v = np.sort(f(255) * y.astype(f))
    ok = hi - lo >= C - 1 and bool(np.all(np.isfinite(v)))
    v = np.minimum(np.maximum(v, lo), hi)
    for k in range(1, C):
        v[k] = max(v[k], v[k - 1] + f(1))
    if v[-1] > hi:
        v[-1] = hi
        for k in range(C - 2, -1, -1):
            v[k] = min(v[k], v[k + 1] - f(1))
        ok = ok and not v[0] < lo
    return v.astype(np.float64) if ok else np.full(C, np.nan)


@pytest.mark.parametrize("count", [1, 3, 511, 512, 513, 514, 515])
@pytest.mark.parametrize("C", [2, 5, 8])
def test_starts(count, C):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1601_00072_amd import MLP
    print("CASE starts", count, "C", C, flush=True)
    rng = np.random.default_rng(count * 10 + C)
    lo = rng.integers(0, 250, count)
    width = rng.integers(1, 256, count)  # some too narrow for C centroids
    h = np.zeros((count, 256), np.float32)
    for i in range(count):
        w = min(int(width[i]), 256 - int(lo[i]))
        h[i, lo[i]:lo[i] + w] = rng.random(w).astype(np.float32) + np.float32(0.01)
        h[i] /= h[i].sum()
    h[count // 2, :] = 0.0  # no level at all
    d = torch.from_numpy(h).to("cuda:0")
    with MLP(C, seed=11) as net:
        net.set_params(net.params() + (0.05 * rng.standard_normal(net.n_params)).astype(np.float32))
        y = net.forward(d, bf16=True).cpu().numpy()
        got = net.warm_centroids(d).cpu().numpy()
    want = np.stack([_post(y[i], h[i], C) for i in range(count)])
    assert np.array_equal(got, want, equal_nan=True)
