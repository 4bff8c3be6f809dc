"""Surrogate network at the edges of its tiles: 8 or 16 samples per group with tangents, one or two tiles
of 16 for values alone, 16 samples per workgroup and chunks of 256 or more samples in the backward
pass, unaligned weights.  Against the FP64 oracle; bars as for the other tests of these kernels (FP32
rounding of a 35 590-weight network): 1e-5 forward and Jacobian, 1e-4 gradients.
"""
import numpy as np
import pytest

from helpers import rel_err
from oracle import mlp
from test_gpu_mlp import _params, to_lib

pytestmark = pytest.mark.gpu


def _data(n, offset):
    import torch
    p = _params()
    rng = np.random.default_rng(n)
    x = rng.normal(size=(n, 13)).astype(np.float32).astype(np.float64)
    t = rng.normal(size=(n, 6)).astype(np.float32).astype(np.float64)
    dev = lambda a: torch.tensor(a, dtype=torch.float32, device="cuda")  # noqa: E731
    w = to_lib(p)
    W = torch.cat([torch.zeros(offset, device="cuda"), dev(w)])[offset:]
    return p, x, t, W, dev(x), dev(t)


@pytest.mark.parametrize("n", [7, 8, 9, 16, 17, 2048, 2049, 8200])
def test_tangent_groups(n):
    from paper_2604_22087_amd import fe
    print(f"[mlp tangent] n={n}", flush=True)
    p, x, _, W, xt, _ = _data(n, n % 3)
    y, jac, cache = fe.mlp_forward(W, xt, jacobian=True, cache=True)
    y_ref, c_ref = mlp.forward(p, x)
    assert rel_err(y.double().cpu().numpy(), y_ref) <= 1e-5
    keep = np.r_[0:min(n, 64), max(0, n - 64):n]
    assert rel_err(jac.double().cpu().numpy()[keep], mlp.jacobian(p, x[keep])) <= 1e-5
    for layer in range(3):
        assert rel_err(cache.double().cpu().numpy()[:, layer], c_ref["zs"][layer]) <= 1e-5


@pytest.mark.parametrize("n", [1, 15, 16, 33, 255, 257, 8192, 8193, 16385, 20001])
def test_training_tiles(n):
    from paper_2604_22087_amd import fe
    print(f"[mlp training] n={n}", flush=True)
    p, x, t, W, xt, tt = _data(n, n % 3)
    y, _, cache = fe.mlp_forward(W, xt, cache=True)
    y_ref, c_ref = mlp.forward(p, x)
    assert rel_err(y.double().cpu().numpy(), y_ref) <= 1e-5
    for layer in range(3):
        assert rel_err(cache.double().cpu().numpy()[:, layer], c_ref["zs"][layer]) <= 1e-5
    dW, loss = fe.mlp_backward(W, xt, cache, y, tt)
    grads = mlp.backward(p, c_ref, y_ref, t)
    g_ref = np.concatenate([np.concatenate([gW.T.ravel(), gb]) for gW, gb in grads])
    assert rel_err(dW.double().cpu().numpy(), g_ref) <= 1e-4
    assert float(loss) == pytest.approx(mlp.mse_loss(y_ref, t), rel=1e-5)
