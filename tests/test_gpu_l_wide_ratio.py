"""The row gather of an L-shaped domain where more than 3 subdomains cover a point along an axis (width
ratios of 3 and more: its general loop, which skips the discarded subdomains by the block map), with
and without Dirichlet rows in the same launch, against the oracle's dense matrix.

Tolerance: entries of both sides agree to a few ulp, so the products agree to 1e-12 of the norm."""
import dataclasses

import numpy as np
import pytest

from inputs import configs, feature_params
from inputs.problems import grid_points
from oracle import assemble as asm
from oracle import geometry as geo

from gpu_util import dev, torch_mod

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("delta", [2.9, 3.1, 4.2, 6.5])
@pytest.mark.parametrize("nb", [0, 3, 16, 40])
def test_products(delta, nb):
    from paper_2409_01949_amd import Problem
    torch = torch_mod()
    K = 5
    spec = dataclasses.replace(configs.helmholtz(omega=2.0, levels=((1, 1), (5, 6), (9, 8)), K=K, n=31), delta=delta)
    Wf, bf = feature_params(spec)
    xb = configs.boundary_points(spec)[:nb]
    bc = dict(bc_pts=xb, bc_vals=configs.exact(spec, xb), bc_weight=3.0) if nb else {}
    P = Problem.from_spec(spec, Wf, bf, "fp64", **bc)
    P.assemble(dev(configs.forcing(spec)))
    W, b = geo.kept_parameters(spec, Wf, bf)
    blocks = asm.assemble_blocks(spec, W, b)
    inside = configs.in_l_shape(spec, grid_points(spec))
    N, n = int(inside.sum()), len(blocks) * K
    M = asm.dense_from_blocks(blocks, N, n)
    if nb:
        M = np.vstack([M, asm.dirichlet_rows(spec, W, b, xb) * (3.0 / asm.dirichlet_weight(spec, nb))])
    rows = np.concatenate([np.nonzero(inside)[0], inside.size + np.arange(nb)])
    rng = np.random.default_rng(nb)
    v, u = rng.standard_normal(n), np.zeros(inside.size + nb)
    u[rows] = rng.standard_normal(rows.size)
    y = torch.empty(u.size, dtype=torch.float64, device="cuda")
    x = torch.empty(n, dtype=torch.float64, device="cuda")
    P.matvec(dev(v), y)
    P.rmatvec(dev(u), x)
    P.destroy()
    yr, xr, yg = M @ v, M.T @ u[rows], y.cpu().numpy()
    assert np.linalg.norm(yg[rows] - yr) <= 1e-12 * np.linalg.norm(yr)
    assert not np.any(yg[:inside.size][~inside])
    assert np.linalg.norm(x.cpu().numpy() - xr) <= 1e-12 * np.linalg.norm(xr)
