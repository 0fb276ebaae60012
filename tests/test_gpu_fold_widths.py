"""The folded matrix M R^-1 at the edges of its kernels: column counts around the 16-feature tiles
and the 32, 64, 128 and 256 columns of the layouts, blocks of a few points up to several runs of
256 with odd ends (points are stored in pairs), every stored precision.

The FP64 fold against the oracle within fold_tolerance; the low-precision copy is the rounding of
the device's own FP64 fold, exactly."""
import numpy as np
import pytest

from inputs import configs
from oracle import assemble as asm
from oracle import linalg, lowprec

from gpu_util import build, device_blocks, fold_tolerance, torch_mod

pytestmark = pytest.mark.gpu
SHIFT = 1e-3
ROUND = {"fp32": lowprec.to_f32, "bf16": lowprec.to_bf16, "fp16": lowprec.to_fp16}


@pytest.mark.parametrize("store", list(ROUND))
@pytest.mark.parametrize("K", [3, 16, 17, 32, 33, 64, 65, 127, 128, 129, 256])
@pytest.mark.parametrize("n", [21, 401, 1707])
def test_fold(n, K, store):
    torch_mod()
    spec = configs.tiny1d(K=K, J=2, n=n, delta=1.9, seed=n + K)
    P, W, b, _ = build(spec, store_prec=store)
    blocks = asm.assemble_blocks(spec, W, b)
    assert P.precondition(SHIFT) == 0
    fold = linalg.fold_blocks(blocks, linalg.block_jacobi_factors(blocks, SHIFT))
    hi, lo = device_blocks(P, K, "fp64", folded=True), device_blocks(P, K, store, folded=True)
    P.destroy()
    for (_, h), (_, q), ref in zip(hi, lo, fold):
        assert np.abs(h - ref.M).max() <= fold_tolerance(ref.M, K, SHIFT)
        assert np.array_equal(q, ROUND[store](h))
