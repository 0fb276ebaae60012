"""MLP products at the edges of their tiles (64 x 64 outputs, stages of 128 in k with three loaded
ahead, column sums over 256 rows), for operands whose rows allow 16-byte loads and for odd widths:
a network of one layer, whose outputs and gradients are plain sums of products of known bfloat16
numbers.

Tolerance: an FP32 sum of n products differs from the exact one by at most (n + 2) 2^-24 of the sum
of their magnitudes."""
import numpy as np
import pytest

from inputs import mlp_init
from oracle import lowprec

from gpu_util import torch_mod

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


@pytest.mark.parametrize("n_in,n_out", [(1, 1), (7, 65), (8, 64), (65, 192), (127, 9), (128, 63),
                                        (129, 16), (384, 72), (385, 24), (512, 130), (641, 200)])
@pytest.mark.parametrize("batch", [1, 63, 64, 255, 257, 513, 1500])
def test_one_layer(n_in, n_out, batch):
    torch = torch_mod()
    from paper_2409_01949_amd import MLP
    dims = [n_in, n_out]
    m = MLP(dims, 1500)
    p = mlp_init(dims, n_in + n_out)
    m.set_params(p)
    rng = np.random.default_rng(batch)
    X = rng.standard_normal((batch, n_in)).astype(np.float32)
    T = rng.standard_normal((batch, n_out)).astype(np.float32)
    xd, td = torch.as_tensor(X).cuda(), torch.as_tensor(T).cuda()
    y = m.forward(xd).cpu().numpy()
    loss = m.train_step(xd, td, update=False)
    g = m.get_grads().astype(np.float64)
    m.destroy()
    W, b = p[:n_in * n_out].reshape(n_out, n_in), p[n_in * n_out:]
    Xb, Wb = lowprec.to_bf16(X.astype(np.float64)), lowprec.to_bf16(W.astype(np.float64))
    ref, mag = Xb @ Wb.T + b, np.abs(Xb) @ np.abs(Wb.T) + np.abs(b)
    assert np.all(np.abs(y - ref) <= (n_in + 2) * U * mag)
    d = y - T
    G = lowprec.to_bf16((np.float32(2.0) / np.float32(d.size) * d).astype(np.float64))
    dW, db = g[:n_in * n_out].reshape(n_out, n_in), g[n_in * n_out:]
    assert np.all(np.abs(dW - G.T @ Xb) <= (batch + 2) * U * (np.abs(G).T @ np.abs(Xb)))
    assert np.all(np.abs(db - G.sum(0)) <= (batch + 2) * U * np.abs(G).sum(0))
    assert abs(loss - np.mean(d.astype(np.float64) ** 2)) <= 1e-12 * loss
