"""The two launches of a training step at the edges of their splits: odd row
counts (two rows per block), the 128-row chunks of the gradient sums, every
output width, and inputs that are only 4-byte aligned -- loss and gradient
against the FP64 oracle (bounds as for the network's other gradients)."""
import numpy as np
import pytest

from oracle import mlp_ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 2, 3, 127, 128, 129, 255, 257])
@pytest.mark.parametrize("C", [2, 5, 8])
def test_rows(rows, C):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1601_00072_amd import MLP
    print("CASE train step rows", rows, "C", C, flush=True)
    rng = np.random.default_rng(rows * 10 + C)
    X = rng.gamma(0.3, size=(rows, 256))
    X = (X / X.sum(axis=1, keepdims=True)).astype(np.float32)
    T = rng.uniform(0.0, 1.0, size=(rows, C)).astype(np.float32)
    buf = torch.zeros(rows * 256 + 4, dtype=torch.float32, device="cuda:0")
    Xd = buf[1:1 + rows * 256].view(rows, 256)
    Xd.copy_(torch.from_numpy(X))
    Td = torch.from_numpy(T).to("cuda:0")
    with MLP(C, seed=7) as net:
        theta = net.params() + (0.02 * rng.standard_normal(net.n_params)).astype(np.float32)
        net.set_params(theta)
        loss, g = net.loss_grad(Xd, Td)
        again, g2 = net.loss_grad(Xd, Td)
        before = net.params()
        net.train(Xd, Td, epochs=1, batch=rows, lr=1e-3)
        after = net.params()
    assert loss == again and np.array_equal(g, g2) and np.array_equal(before, theta)
    th, Xf, Tf = theta.astype(np.float64), X.astype(np.float64), T.astype(np.float64)
    assert abs(loss - mlp_ref.loss(th, Xf, Tf, C)) <= 1e-5 * mlp_ref.loss(th, Xf, Tf, C)
    ref = mlp_ref.grad(th, Xf, Tf, C)
    for a, b in zip(mlp_ref.unpack(g.astype(np.float64), C), mlp_ref.unpack(ref, C)):
        assert np.max(np.abs(a - b)) <= 1e-4 * np.max(np.abs(b)) + 1e-9
    # the first Adam step moves every parameter by lr sign(g) where g stands clear of zero
    clear = np.abs(ref) > 1e-5
    moved = after.astype(np.float64) - theta
    assert np.max(np.abs(moved[clear] + 1e-3 * np.sign(ref[clear]))) <= 1e-3 * 2e-3


@pytest.mark.parametrize("sizes", [[1], [16384], [16385], [5, 70000, 131072, 1], [4096] * 600, [40000] * 70])
def test_histogram_splits(sizes):
    """Counts of one and of several blocks per instance, against numpy."""
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1601_00072_amd import histogram
    print("CASE histogram", len(sizes), sizes[:4], flush=True)
    rng = np.random.default_rng(len(sizes))
    x = rng.integers(0, 256, sum(sizes) + 3, dtype=np.uint8)
    x[: x.size // 2] = 0
    got = histogram(torch.from_numpy(x).to("cuda:0")[3:], sizes).cpu().numpy()
    off = 3
    for g, n in zip(got, sizes):
        want = np.bincount(x[off:off + n], minlength=256).astype(np.float64) / n
        assert np.array_equal(g, want.astype(np.float32))
        off += n


@pytest.mark.parametrize("count", [1, 511, 512, 513, 515])
def test_inference_splits(count):
    """One and four histograms per block give the same bits, row by row."""
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1601_00072_amd import MLP
    print("CASE inference count", count, flush=True)
    h = torch.rand(count, 256, device="cuda:0")
    h[:, 200:] = 0
    h /= h.sum(dim=1, keepdim=True)
    with MLP(4, seed=2) as net:
        y = net.forward(h, bf16=True)
        for i in {0, count // 2, count - 1}:
            assert torch.equal(y[i:i + 1], net.forward(h[i:i + 1], bf16=True))
            assert torch.equal(net.warm_centroids(h)[i], net.warm_centroids(h[i:i + 1])[0])
