"""Batches whose subdomains outnumber the grid points, so that supports hold no point at all: such a
block has no rows, its Gram block is zero and its factor the identity, for subdomain blocks and for
patches of them (up to 280 columns: squares of outputs off the diagonal too).  Preconditioned LSQR
iterates against the oracle's, at the 1e-8 of the other block-Jacobi iterate tests."""
import dataclasses

import numpy as np
import pytest

from inputs import configs
from oracle import linalg

from gpu_util import torch_mod
from test_gpu_patches import R, _coefs, _make

pytestmark = pytest.mark.gpu
SHIFT = 1e-2


@pytest.mark.parametrize("K", [5, 70])
@pytest.mark.parametrize("patch", [1, 2])
def test_preconditioned_batch(patch, K):
    torch = torch_mod()
    specs = [configs.tiny1d(K=K, J=40, n=13, delta=1.9, seed=K),
             dataclasses.replace(configs.small2d(seed=K), n_points=(6, 7), levels=((1, 1), (31, 33)), K=K)]
    B, oracle = _make("fp64", specs)
    blocks = [linalg.patch_blocks(bl, patch) for _, bl, _ in oracle]
    assert all(any(p.rows.size == 0 for p in pbs) for pbs in blocks)
    # the identity: these, and blocks whose only point is a corner, where the hard constraint and
    # its first derivatives vanish
    zero = sum(not p.M.any() for pbs in blocks for p in pbs)
    try:
        assert B.precondition(SHIFT, patch=patch) == zero
        coef = torch.empty(R * B.sizes["n_phi"], dtype=torch.float64, device="cuda")
        B.solve(coef, iter_lim=2, atol=0.0, btol=0.0, check_every=2, precond=True)
        got = _coefs(B, coef, oracle)
    finally:
        B.destroy()
    for (s, bl, h), pbs, x in zip(oracle, blocks, got):
        facs = linalg.block_jacobi_factors(pbs, SHIFT)
        fold = linalg.fold_blocks(pbs, facs)
        for j in range(R):
            res = linalg.lsqr(lambda y: linalg.patch_matvec(fold, y, s.n_rows),
                              lambda u: linalg.patch_rmatvec(fold, u), h[j], len(bl) * s.K,
                              atol=0, btol=0, iter_lim=2)
            ref = linalg.patch_recover(pbs, facs, res.x)
            assert np.linalg.norm(x[j] - ref) <= 1e-8 * np.linalg.norm(ref)
