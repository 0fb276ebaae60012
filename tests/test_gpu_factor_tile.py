"""Block-Jacobi factors of narrow blocks, one wavefront each: at the edges of its widths (4, 16 and 24
columns) and of the rule that keeps it (up to 1,024 blocks above 16 columns), and the Gram blocks on
squares of 32 and 64 columns, against the oracle; failed and all-zero blocks.

Tolerance: fold_tolerance, as for the wider blocks."""
import dataclasses

import numpy as np
import pytest

from inputs import configs, feature_params
from oracle import assemble as asm
from oracle import linalg

from gpu_util import build, dev, device_blocks, fold_tolerance, torch_mod

pytestmark = pytest.mark.gpu
SHIFT = 1e-4


def check(blocks, got, K):
    fold = linalg.fold_blocks(blocks, linalg.block_jacobi_factors(blocks, SHIFT))
    for ref, m in zip(fold, got):
        assert np.abs(m - ref.M).max() <= fold_tolerance(ref.M, K, SHIFT)


def batch_blocks(B, K):
    torch = torch_mod()
    out = torch.empty(B.sizes["nnz"], dtype=torch.float64, device="cuda")
    table = B.copy_blocks(out, "fp64", folded=True)
    host = out.cpu().numpy()
    for row in table:
        n, off = int(row[3] * row[5]), int(row[7])
        yield host[off:off + n * K].reshape(K, n).T


@pytest.mark.parametrize("K", [3, 4, 5, 16, 17, 24, 25, 32, 33, 64, 65])
def test_widths(K):
    from paper_2409_01949_amd import Batch
    spec = configs.tiny1d(K=K, J=5, n=700, delta=1.9, seed=K)
    P, W, b, f = build(spec)
    blocks = asm.assemble_blocks(spec, W, b)
    assert P.precondition(SHIFT) == 0
    check(blocks, [m for _, m in device_blocks(P, K, "fp64", folded=True)], K)
    P.destroy()
    B = Batch([spec], [W], [b], 1)
    B.assemble(dev(f))
    assert B.precondition(SHIFT) == 0
    check(blocks, batch_blocks(B, K), K)
    B.destroy()


@pytest.mark.parametrize("K", [16, 20])
@pytest.mark.parametrize("J", [(32, 32), (25, 41)])
def test_many_blocks(J, K):
    from paper_2409_01949_amd import Batch
    spec = dataclasses.replace(configs.small2d(), n_points=(70, 90), levels=(J,), K=K, w_range=(-1.0, 1.0))
    W, b = feature_params(spec)
    B = Batch([spec], [W], [b], 1)
    B.assemble(dev(configs.forcing(spec)))
    assert B.precondition(SHIFT) == 0
    check(asm.assemble_blocks(spec, W, b), batch_blocks(B, K), K)
    B.destroy()


@pytest.mark.parametrize("K", [3, 12, 20])
def test_singular_and_zero_blocks(K):
    """Equal columns factor with the shift (and its retries), a zero block is the identity."""
    spec = configs.tiny1d(K=K, J=3, n=200, delta=1.9)
    W, b = feature_params(spec)
    W[:K], b[:K] = 0.0, 0.5
    W[2 * K:], b[2 * K:] = 0.0, 0.0
    from paper_2409_01949_amd import Batch, Problem
    P = Problem.from_spec(spec, W, b)
    P.assemble(dev(configs.forcing(spec)))
    assert P.precondition(1e-12) == 0
    got = [m for _, m in device_blocks(P, K, "fp64", folded=True)]
    P.destroy()
    B = Batch([spec], [W], [b], 1)
    B.assemble(dev(configs.forcing(spec)))
    assert B.precondition(1e-12) == 1      # batches count the zero block
    both = [got, list(batch_blocks(B, K))]
    B.destroy()
    for blocks in both:
        assert np.all(blocks[2] == 0.0)
        for m in blocks[:2]:
            assert np.all(np.isfinite(m)) and np.linalg.norm(m, axis=0).max() <= 1.0 + 1e-3
