"""Gram blocks at the edges of the kernel's squares (32, 64, 96 and 128 columns, several squares),
of its 16 x 16 tiles and of its masked loads (odd grid heights, one-point overlaps), every stored
precision, all pairs and diagonal blocks, against the oracle.

Tolerances: FP64 1e-12, the narrow copies 1e-5 (FP32 accumulation over at most 2,500 points), of
the block's largest sum of |products|: what a rounded sum's error is proportional to (a one-column
block's own entry can cancel to nothing)."""
import dataclasses

import numpy as np
import pytest

from inputs import configs
from oracle import assemble as asm
from oracle import geometry as geo
from oracle import linalg

from gpu_util import build, device_blocks, torch_mod

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store", ["fp64", "fp32", "bf16", "fp16"])
@pytest.mark.parametrize("K", [1, 15, 16, 17, 33, 48, 64, 65, 80, 96, 97, 128, 129, 161, 256])
@pytest.mark.parametrize("which", ["all", "diag"])
def test_gram(K, store, which):
    torch = torch_mod()
    spec = dataclasses.replace(configs.small2d(seed=K), n_points=(31, 43), K=K, w_range=(-1.0, 1.0),
                               levels=((1, 1), (2, 3)) if K > 64 else ((1, 1), (3, 2), (7, 9)))
    P, W, b, _ = build(spec, store_prec=store)
    # the oracle's products of the device's own stored entries
    blocks = [dataclasses.replace(blk, M=M) for blk, (_, M) in
              zip(asm.assemble_blocks(spec, W, b), device_blocks(P, K, store))]
    pairs = geo.overlap_pairs(spec, [blk.rows for blk in blocks])
    if which == "diag":
        pairs = [p for p in pairs if p[0] == p[1]]
    ref = linalg.gram_blocks(blocks, pairs)
    scale = linalg.gram_blocks([dataclasses.replace(blk, M=np.abs(blk.M)) for blk in blocks], pairs)
    P.gram(store, which)
    G = torch.empty(len(pairs) * K * K, dtype=torch.float64 if store == "fp64" else torch.float32,
                    device="cuda")
    table = P.copy_gram(G)
    host = G.double().cpu().numpy().reshape(-1, K, K)
    P.destroy()
    assert {(int(i), int(j)) for i, j, _ in table} == set(ref)
    tol = 1e-12 if store == "fp64" else 1e-5
    for (i, j, o) in table:
        key = (int(i), int(j))
        assert np.abs(host[o // (K * K)] - ref[key]).max() <= tol * scale[key].max()
