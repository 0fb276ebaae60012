"""MLP products over few k (stages of 32 up to 64 of them) and few rows (elements stored one by one
below 64): one layer against plain sums as for the longer products, and hidden layers against the
same rows in a longer batch, which go through the whole-row stores.

Forward rows do not depend on the batch, bit for bit.  Gradients of the rows taken 2^r times are those
of the rows (the mean divides each summand, exactly in binary), up to the FP32 sum of at most 128 terms:
2 x 130 x 2^-24 = 1.6e-5 of the sum of magnitudes, which the cancellation of these random sums (a
factor of the order sqrt(64)) brings to at most 2e-4 of the norm."""
import numpy as np
import pytest

from inputs import mlp_init

from gpu_util import torch_mod
from test_gpu_mlp_tiles import test_one_layer as one_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_in,n_out", [(2, 16), (31, 17), (32, 64), (33, 8), (40, 65), (63, 15), (64, 16), (65, 70), (66, 1)])
@pytest.mark.parametrize("batch", [2, 15, 16, 31, 32, 33, 62, 65, 66])
def test_one_short_layer(n_in, n_out, batch):
    one_layer(n_in, n_out, batch)


@pytest.mark.parametrize("dims", [[4, 16, 16, 8], [40, 62, 13, 96, 6], [64, 64, 64], [33, 5, 70, 3], [7, 1, 24]])
@pytest.mark.parametrize("batch", [1, 16, 40, 63])
def test_hidden_layers(dims, batch):
    torch = torch_mod()
    from paper_2409_01949_amd import MLP
    m = MLP(dims, 128)
    m.set_params(mlp_init(dims, sum(dims)))
    rng = np.random.default_rng(batch)
    X = torch.as_tensor(rng.standard_normal((128, dims[0])).astype(np.float32)).cuda()
    T = torch.as_tensor(rng.standard_normal((128, dims[-1])).astype(np.float32)).cuda()
    assert torch.equal(m.forward(X)[:batch], m.forward(X[:batch].contiguous()))
    m.train_step(X[:batch].contiguous(), T[:batch].contiguous(), update=False)
    g = m.get_grads().astype(np.float64)
    reps = {1: 128, 16: 8}.get(batch, 2)      # to 64 rows or more
    m.train_step(X[:batch].repeat(reps, 1), T[:batch].repeat(reps, 1), update=False)
    g2 = m.get_grads().astype(np.float64)
    m.destroy()
    assert np.linalg.norm(g2 - g) <= 2e-4 * np.linalg.norm(g)
