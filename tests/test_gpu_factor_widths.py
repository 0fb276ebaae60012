"""The block-Jacobi factors at the edges of their panels (16 and 32 rows) and of the wavefront
layouts (128, 256 and 512 columns), against the oracle: R^-1 through the folded matrix M R^-1 and
through x = R^-1 y, for single problems, batches and patches; failed factorisations and all-zero
blocks.

Tolerance: fold_tolerance, the shift-scaled bound of the fold tests (the rounding of the Gram
block, of condition K/shift, times a margin of 4)."""
import dataclasses

import numpy as np
import pytest

from inputs import configs, feature_params
from oracle import assemble as asm
from oracle import linalg

from gpu_util import build, dev, device_blocks, fold_tolerance, torch_mod
from test_gpu_patches import _check_patches, _make

pytestmark = pytest.mark.gpu
SHIFT = 1e-4


@pytest.mark.parametrize("K", [1, 2, 15, 16, 17, 31, 32, 33, 48, 63, 65, 100, 127, 128, 129, 144,
                               160, 191, 255, 256])
def test_single(K):
    torch = torch_mod()
    spec = configs.tiny1d(K=K, J=3, n=600, delta=1.9, seed=K)
    P, W, b, f = build(spec)
    blocks = asm.assemble_blocks(spec, W, b)
    assert P.precondition(SHIFT) == 0
    fold = linalg.fold_blocks(blocks, linalg.block_jacobi_factors(blocks, SHIFT))
    for (_, got), ref in zip(device_blocks(P, K, "fp64", folded=True), fold):
        assert np.abs(got - ref.M).max() <= fold_tolerance(ref.M, K, SHIFT)
    # one preconditioned LSQR step returns x = R^-1 y: M x is the folded matrix's y in its rows
    coef = torch.empty(P.sizes["n_phi"], dtype=torch.float64, device="cuda")
    y = torch.empty(600, dtype=torch.float64, device="cuda")
    P.solve(coef, method="lsqr", precond=True, iter_lim=1, atol=0.0, btol=0.0)
    P.matvec(coef, y)
    P.destroy()
    n = coef.numel()
    one = linalg.lsqr(lambda v: asm.matvec(fold, v, 600), lambda r: asm.rmatvec(fold, r, n),
                      asm.rhs(spec, f), n, atol=0, btol=0, iter_lim=1)
    ref = asm.matvec(fold, one.x, 600)
    tol = max(fold_tolerance(q.M, K, SHIFT) / np.abs(q.M).max() for q in fold)
    assert np.linalg.norm(y.cpu().numpy() - ref) <= 10 * tol * np.linalg.norm(ref)


@pytest.mark.parametrize("K", [1, 5, 16, 31, 33, 64, 65, 97, 128])
@pytest.mark.parametrize("patch", [1, 2, 4])
def test_batch(K, patch):
    if patch * K > 512:      # 1D: a patch holds `patch` subdomains
        pytest.skip("wider than 512 columns")
    specs = [dataclasses.replace(configs.tiny1d(K=k, J=5, n=700, delta=1.9, seed=k),
                                 meta={"family": "ode_cos", "omega": 3.0}) for k in (K, max(1, K - 7))]
    B, oracle = _make("fp64", specs)
    if patch == 1:
        assert B.precondition(SHIFT) == 0
        torch = torch_mod()
        out = torch.empty(B.sizes["nnz"], dtype=torch.float64, device="cuda")
        table = B.copy_blocks(out, "fp64", folded=True)
        host = out.cpu().numpy()
        k = 0
        for s, bl, _ in oracle:
            for ref in linalg.fold_blocks(bl, linalg.block_jacobi_factors(bl, SHIFT)):
                n, off = int(table[k][3] * table[k][5]), int(table[k][7])
                got = host[off:off + n * s.K].reshape(s.K, n).T
                assert np.abs(got - ref.M).max() <= fold_tolerance(ref.M, s.K, SHIFT)
                k += 1
    else:
        _check_patches(B, oracle, patch, "fp64", SHIFT)
    B.destroy()


@pytest.mark.parametrize("K", [5, 40, 130])
def test_singular_and_zero_blocks(K):
    """Zero weights make every feature of a block the same column (rank one: the shifted Gram block
    still factors, with retries where rounding makes it indefinite), zero weights and biases make
    the block zero (the identity)."""
    spec = configs.tiny1d(K=K, J=3, n=200, delta=1.9)
    W, b = feature_params(spec)
    W[:K] = 0.0
    b[:K] = 0.5
    W[2 * K:] = 0.0
    b[2 * K:] = 0.0
    from paper_2409_01949_amd import Problem
    P = Problem.from_spec(spec, W, b)
    P.assemble(dev(configs.forcing(spec)))
    assert P.precondition(1e-12) == 0
    got = [m for _, m in device_blocks(P, K, "fp64", folded=True)]
    P.destroy()
    assert np.all(got[2] == 0.0)
    for m in got[:2]:
        assert np.all(np.isfinite(m))
        # columns of M R^-1 have norm at most 1, up to the rounding of the shifted factor
        assert np.linalg.norm(m, axis=0).max() <= 1.0 + 1e-3
