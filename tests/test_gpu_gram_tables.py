"""The Gram launch tables, dealt to the XCDs by second block, from a few chunks to more than run at
once, and made anew on one handle as the precision and the kind of blocks alternate, against the
oracle.

Tolerances as for the widths: 1e-12 in FP64, 1e-5 in FP32, of the largest sum of |products|."""
import dataclasses

import numpy as np
import pytest

from inputs import configs
from oracle import assemble as asm
from oracle import geometry as geo
from oracle import linalg

from gpu_util import build, device_blocks, torch_mod

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels", [((2, 2),), ((13, 13),), ((14, 14),), ((1, 1), (6, 6), (12, 12))])
def test_alternating(levels):
    torch = torch_mod()
    K = 3
    spec = dataclasses.replace(configs.small2d(), n_points=(61, 58), K=K, w_range=(-1.0, 1.0), levels=levels)
    P, W, b, _ = build(spec, store_prec="fp32")
    ref = {}
    for prec in ("fp64", "fp32"):
        blocks = [dataclasses.replace(blk, M=M) for blk, (_, M) in
                  zip(asm.assemble_blocks(spec, W, b), device_blocks(P, K, prec))]
        pairs = geo.overlap_pairs(spec, [blk.rows for blk in blocks])
        ref[prec] = (linalg.gram_blocks(blocks, pairs), linalg.gram_blocks(
            [dataclasses.replace(blk, M=np.abs(blk.M)) for blk in blocks], pairs))
    for prec, which in [("fp64", "all"), ("fp32", "all"), ("fp64", "all"), ("fp32", "diag"),
                        ("fp64", "diag"), ("fp32", "all")]:
        keys = [p for p in pairs if which == "all" or p[0] == p[1]]
        P.gram(prec, which)
        G = torch.empty(len(keys) * K * K, device="cuda",
                        dtype=torch.float64 if prec == "fp64" else torch.float32)
        table = P.copy_gram(G)
        host = G.double().cpu().numpy().reshape(-1, K, K)
        assert [(int(i), int(j)) for i, j, _ in table] == sorted(keys)
        tol = 1e-12 if prec == "fp64" else 1e-5
        for i, j, o in table:
            g, scale = (r[(int(i), int(j))] for r in ref[prec])
            assert np.abs(host[o // (K * K)] - g).max() <= tol * scale.max()
    P.destroy()
