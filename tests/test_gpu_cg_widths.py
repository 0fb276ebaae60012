"""Preconditioned CG on the Gram blocks at the edges of its step's kernels: blocks around the groups
of 32 features and the 64 and 128 features of the layouts, one above them (separate kernels), and
more blocks than workgroups.

Tolerance as in the CG tests: the iterates agree with the oracle's within max(1e-9, 50 times the
oracle's own spread when its factors come from row-permuted blocks)."""
import dataclasses

import numpy as np
import pytest

from inputs import configs
from oracle import assemble as asm
from oracle import geometry as geo
from oracle import linalg

from gpu_util import build, torch_mod

pytestmark = pytest.mark.gpu
SHIFT = 1e-2


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("K,levels", [(K, ((1, 1), (2, 3))) for K in
                                      (1, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129)]
                         + [(3, ((1, 1), (34, 32)))])
def test_iterates(K, levels):
    torch = torch_mod()
    spec = dataclasses.replace(configs.small2d(seed=K), K=K, levels=levels, w_range=(-1.0, 1.0))
    P, W, b, f = build(spec)
    blocks = asm.assemble_blocks(spec, W, b)
    n = P.sizes["n_phi"]
    G = linalg.gram_blocks(blocks, geo.overlap_pairs(spec, [blk.rows for blk in blocks]))
    g = asm.rmatvec(blocks, asm.rhs(spec, f), n)
    rng = np.random.default_rng(K)
    perm = [rng.permutation(blk.M.shape[0]) for blk in blocks]
    alt = [asm.Block(blk.sd, blk.rows[p], blk.M[p]) for blk, p in zip(blocks, perm)]
    facs, facs_alt = (linalg.block_jacobi_factors(x, SHIFT) for x in (blocks, alt))
    assert P.precondition(SHIFT) == 0
    P.gram("fp64", "all")
    for k in (1, 4):
        coef = torch.empty(n, dtype=torch.float64, device="cuda")
        info = P.solve(coef, method="normal_cg", precond=True, iter_lim=k, atol=0, btol=0,
                       check_every=k)
        ref, two = (linalg.normal_pcg(lambda p: linalg.gram_apply(G, blocks, p), g, k,
                                      apply_Minv=lambda r, F=F: linalg.block_jacobi_inverse_apply(
                                          blocks, F, r)) for F in (facs, facs_alt))
        assert info["iters"] == k
        assert _rel(coef.cpu().numpy(), ref) <= max(1e-9, 50 * _rel(two, ref))
    P.destroy()
