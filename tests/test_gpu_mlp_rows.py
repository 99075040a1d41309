"""The network's kernels at the edges of their row tiles (1, 4, 8 and 16 rows per
workgroup, groups of 16 rows in the gradient), against the FP64 oracle at the
tolerances of test_gpu_mlp.py, and the independence of the tiling: every product is a
chain in the order of its terms, so a row's outputs do not depend on the rows it is
computed with (bitwise)."""
import numpy as np
import pytest

from oracle import mlp_oracle as M
from tests.test_gpu_mlp import _blocks, _data

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0911_0459_amd import lbcap
    return lbcap


@pytest.mark.parametrize("n", [3, 4, 5, 256, 257, 1024, 1025, 2048, 2049, 2065])
def test_forward_at_tile_edges(L, n):
    net = L.MLP(seed=31)
    X, _ = _data(n, seed=n)
    y = net.predict(X)
    ref = M.forward(net.get_params().astype(np.float64), X.astype(np.float64))
    assert np.abs(y - ref).max() <= 2e-5 * np.abs(ref).max()
    some = [0, n // 2, n - 1]
    for r in some:
        assert np.array_equal(net.predict(X[r:r + 1])[0], y[r]), r


@pytest.mark.parametrize("n", [1, 15, 16, 17, 1024, 1025, 2100])
def test_gradient_at_tile_edges(L, n):
    net = L.MLP(seed=32)
    X, Y = _data(n, seed=n)
    loss, g = net.loss_grad(X, Y)
    loss_o, g_o = M.loss_grad(net.get_params().astype(np.float64), X.astype(np.float64), Y.astype(np.float64))
    assert abs(loss - loss_o) <= 1e-5 * loss_o
    for lo, hi in _blocks():
        assert np.abs(g[lo:hi] - g_o[lo:hi]).max() <= 1e-4 * np.abs(g_o[lo:hi]).max(), (lo, hi)


def test_weights_follow_training_and_setting(L):
    """The forward pass multiplies packed copies of the weights: after training steps
    and after set_params they are those of get_params."""
    X, Y = _data(40, seed=3)
    a, b = L.MLP(seed=33), L.MLP(seed=34)
    a.train(X, Y, epochs=3, batch=17, lr=1e-2, seed=1)
    p = a.get_params()
    ref = M.forward(p.astype(np.float64), X.astype(np.float64))
    assert np.abs(a.predict(X) - ref).max() <= 2e-5 * np.abs(ref).max()
    b.set_params(p)
    assert np.array_equal(a.predict(X), b.predict(X))
    for u, v in zip(a.loss_grad(X, Y), b.loss_grad(X, Y)):
        assert np.array_equal(u, v)


def test_output_that_overlaps_the_inputs(L):
    """predict_device_noalloc reads every row of X before it overwrites any."""
    import torch
    net = L.MLP(seed=35)
    n = 900
    X, _ = _data(n, seed=4)
    buf = torch.zeros(n * 64 + 64, device="cuda")
    x = buf[64:64 + n * 19].view(n, 19)
    x.copy_(torch.from_numpy(X))
    torch.cuda.synchronize()
    y = buf[:n * 64].view(n, 64)
    net.predict_device_noalloc(x, y)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), net.predict(X))
