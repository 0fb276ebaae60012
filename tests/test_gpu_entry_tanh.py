"""The feature kernels' tanh and the rounding of the stored copies, entry by entry.

An identity problem with one subdomain on [-1, 1], no constraint and weights 2^j, zero biases has
entries tanh(2^j x) / sqrt(N) with x the grid point: with N a power of 4 the scale is a power of
two, and 2^j x + 0 is exact, so an entry is the device's tanh of a known double times an exact
factor.  The table method's error is at most 0.61 ulp by construction (half a rounding, plus the
roundings of terms at most 1/64 of the result); tested to 0.75."""
import numpy as np
import pytest

from inputs.problems import ProblemSpec, grid_axes
from oracle import lowprec

from gpu_util import dev, device_blocks

pytestmark = pytest.mark.gpu

ROUND = {"fp32": lowprec.to_f32, "bf16": lowprec.to_bf16, "fp16": lowprec.to_fp16}


@pytest.mark.parametrize("store", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("exponents", [(-140, -60, -30, -24), (-18, -14, -9, -7), (-6, -5, -4, -3),
                                       (-2, -1, 0, 1), (2, 3, 4, 6)])
def test_tanh_and_rounding(store, exponents):
    from paper_2409_01949_amd import Problem
    n, K = 4096, len(exponents)
    spec = ProblemSpec(name="tanh", dim=1, op="identity", ansatz="none", ansatz_omega=0.0,
                       lo=(-1.0,), hi=(1.0,), n_points=(n,), levels=((1,),), delta=1.5, K=K)
    W = 2.0 ** np.asarray(exponents, dtype=np.float64)[:, None]
    P = Problem.from_spec(spec, W, np.zeros(K), store)
    P.assemble(dev(np.zeros(n)))
    (_, got), = device_blocks(P, K, "fp64")
    (_, low), = device_blocks(P, K, store)
    P.destroy()
    x = grid_axes(spec)[0]
    for k in range(K):
        ref = np.tanh((W[k, 0] * x).astype(np.longdouble))
        ulp = np.spacing(np.abs(ref.astype(np.float64)))
        err = np.abs(((got[:, k] * np.sqrt(n)).astype(np.longdouble) - ref) / ulp)
        assert float(err.max()) <= 0.75
    assert np.array_equal(low, ROUND[store](got))
