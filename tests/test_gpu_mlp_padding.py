"""The rows that fill up the last group of 16 in a gradient pass take no part in it: not
even where the biases alone, without a row's inputs, overflow in the second layer."""
import numpy as np
import pytest

from oracle import mlp_oracle as M
from tests.test_gpu_mlp import _blocks

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0911_0459_amd import lbcap
    return lbcap


@pytest.mark.parametrize("n", [1, 7, 16, 1025])
def test_rows_that_fill_up_a_group_take_no_part(L, n):
    net = L.MLP(seed=33)
    p = net.get_params()
    layers = M.unpack(np.arange(p.size))
    at = lambda v: v.astype(np.int64)
    p[at(layers[0][0][:, 0])] = -1e25       # the first input, 1 in every row, takes the bias back
    p[at(layers[0][0][:, 1:])] = 0.0
    p[at(layers[0][1])] = 1e25
    p[at(layers[1][0][3])] = 1e15           # what is left of the bias would overflow here
    net.set_params(p)
    rng = np.random.default_rng(n)
    X = np.concatenate([np.ones((n, 1)), rng.normal(size=(n, 18))], axis=1).astype(np.float32)
    Y = rng.normal(0.0, 0.5, (n, 64)).astype(np.float32)
    loss, g = net.loss_grad(X, Y)
    loss_o, g_o = M.loss_grad(p.astype(np.float64), X.astype(np.float64), Y.astype(np.float64))
    assert np.isfinite(g).all() and abs(loss - loss_o) <= 1e-5 * loss_o
    for lo, hi in _blocks():
        assert np.abs(g[lo:hi] - g_o[lo:hi]).max() <= 1e-4 * np.abs(g_o[lo:hi]).max(), (lo, hi)
    # and the same through a step of training
    last = net.train(X, Y, epochs=1, batch=n, lr=1e-3, seed=1)
    assert np.isfinite(last) and np.isfinite(net.get_params()).all()
