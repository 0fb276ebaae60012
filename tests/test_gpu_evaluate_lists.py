"""Evaluation at the edges of its lane layout, against the oracle: feature counts around 64 (the
(block, feature) pairs a wavefront takes at a time), one to five levels (two are searched at once),
width ratios from 1.1 to 6.9 (up to 7 covering subdomains of 11 candidates per axis), axes with a
single subdomain, point counts that leave wavefronts idle, points on the boundary and off the grid.

Tolerance: the sum has at most 49 x 5 x 130 terms, each to a few ulp, so 1e-12 of the vector's norm
as in the evaluation tests of the core cases."""
import numpy as np
import pytest

from inputs import feature_params
from inputs.problems import ProblemSpec
from oracle import evaluate as ev

from gpu_util import dev, torch_mod

pytestmark = pytest.mark.gpu

CASES = [(1, ((3, 2),), 2.9, 5), (7, ((1, 1), (4, 5)), 1.1, 64), (16, ((16, 16),), 2.9, 301),
         (63, ((1, 4), (3, 1), (5, 5)), 2.9, 33), (64, ((9, 8),), 6.9, 17),
         (65, ((2, 2), (8, 9)), 6.9, 3), (130, ((1, 1), (2, 2), (3, 3), (4, 4), (6, 5)), 4.2, 1)]


@pytest.mark.parametrize("K,levels,delta,n", CASES)
@pytest.mark.parametrize("dim", [1, 2])
def test_evaluate(K, levels, delta, n, dim):
    from paper_2409_01949_amd import Problem
    torch = torch_mod()
    spec = ProblemSpec(name="lists", dim=dim, op="d1" if dim == 1 else "neg_laplace",
                       ansatz="tanh_origin" if dim == 1 else "tanh_box", ansatz_omega=5.0,
                       lo=(-0.5, 0.0)[:dim], hi=(1.0, 1.5)[:dim], n_points=(30, 31)[:dim],
                       levels=tuple(J[:dim] for J in levels), delta=delta, K=K,
                       w_range=(-2.0, 2.0), seed=K)
    W, b = feature_params(spec)
    P = Problem.from_spec(spec, W, b)
    rng = np.random.default_rng(n)
    lo, hi = np.asarray(spec.lo), np.asarray(spec.hi)
    pts = lo + (hi - lo) * rng.random((n, dim))
    pts[0] = lo
    pts[-1] = 0.5 * (lo + hi)
    a = rng.standard_normal(P.sizes["n_phi"])
    u = torch.empty(n, dtype=torch.float64, device="cuda")
    P.evaluate(dev(a), dev(pts), u)
    ref = ev.evaluate(spec, W, b, a, pts)
    P.destroy()
    assert np.linalg.norm(u.cpu().numpy() - ref) <= 1e-12 * max(np.linalg.norm(ref), 1e-300)
