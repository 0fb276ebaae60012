"""Batches whose blocks differ in width: every block takes the Gram square that holds it (32, 64 or 128
columns), whatever the widest of the batch; folded blocks against the oracle, at fold_tolerance."""
import dataclasses

import numpy as np
import pytest

from inputs import configs, feature_params
from oracle import assemble as asm
from oracle import linalg

from gpu_util import dev, fold_tolerance, torch_mod

pytestmark = pytest.mark.gpu
SHIFT = 1e-4


@pytest.mark.parametrize("Ks", [(1, 32, 33), (31, 64, 65), (5, 40, 128), (33, 64), (100, 2, 65)])
def test_folded_blocks(Ks):
    from paper_2409_01949_amd import Batch
    torch = torch_mod()
    specs = [dataclasses.replace(configs.small2d(seed=K), n_points=(23, 19 + i), K=K, w_range=(-1.0, 1.0),
                                 levels=((1, 1), (3, 2))) for i, K in enumerate(Ks)]
    feats = [feature_params(s) for s in specs]
    B = Batch(specs, [w for w, _ in feats], [b for _, b in feats], 1)
    B.assemble(dev(np.concatenate([configs.forcing(s) for s in specs])))
    assert B.precondition(SHIFT) == 0
    out = torch.empty(B.sizes["nnz"], dtype=torch.float64, device="cuda")
    rows = iter(B.copy_blocks(out, "fp64", folded=True))
    host = out.cpu().numpy()
    B.destroy()
    for s, (W, b) in zip(specs, feats):
        blocks = asm.assemble_blocks(s, W, b)
        for ref in linalg.fold_blocks(blocks, linalg.block_jacobi_factors(blocks, SHIFT)):
            r = next(rows)
            n, off = int(r[3] * r[5]), int(r[7])
            got = host[off:off + n * s.K].reshape(s.K, n).T
            assert np.abs(got - ref.M).max() <= fold_tolerance(ref.M, s.K, SHIFT)
