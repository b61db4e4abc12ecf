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
