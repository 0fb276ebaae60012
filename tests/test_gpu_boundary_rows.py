"""Products with soft-constraint rows at the edges of their split: one to a few hundred Dirichlet
rows (a wavefront takes every 16th of them, 8 loads at a time), column counts that fill the last
64 or a row's last 512 columns and ones that do not, against the oracle's dense rows.

Tolerance: entries of both sides agree to a few ulp, so the products agree to 1e-12 of the norm."""
import numpy as np
import pytest

from inputs import configs, feature_params
from inputs.problems import grid_points
from oracle import assemble as asm
from oracle import geometry as geo

from gpu_util import dev, torch_mod

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 5, 16, 37])
@pytest.mark.parametrize("nb", [1, 4, 15, 16, 17, 64, 127, 128, 129, 241])
def test_products(nb, K):
    from paper_2409_01949_amd import Problem
    torch = torch_mod()
    spec = configs.helmholtz(omega=2.0, levels=((1, 1), (4, 4), (6, 6)), K=K, n=30)
    Wf, bf = feature_params(spec)
    xb = configs.boundary_points(spec)[:nb]
    inside = configs.in_l_shape(spec, grid_points(spec))
    P = Problem.from_spec(spec, Wf, bf, "fp64", bc_pts=xb, bc_vals=configs.exact(spec, xb),
                          bc_weight=3.0)
    P.assemble(dev(configs.forcing(spec)))
    W, b = geo.kept_parameters(spec, Wf, bf)
    blocks = asm.assemble_blocks(spec, W, b)
    N, n = int(inside.sum()), len(blocks) * K
    B = asm.dirichlet_rows(spec, W, b, xb) * (3.0 / asm.dirichlet_weight(spec, nb))
    M = np.vstack([asm.dense_from_blocks(blocks, N, n), B])
    rows = np.concatenate([np.nonzero(inside)[0], inside.size + np.arange(nb)])
    rng = np.random.default_rng(nb + K)
    v, u = rng.standard_normal(n), np.zeros(inside.size + nb)
    u[rows] = rng.standard_normal(rows.size)
    y = torch.empty(u.size, dtype=torch.float64, device="cuda")
    x = torch.empty(n, dtype=torch.float64, device="cuda")
    P.matvec(dev(v), y)
    P.rmatvec(dev(u), x)
    assert P.sizes["n_bc"] == nb
    P.destroy()
    yr, xr = M @ v, M.T @ u[rows]
    yg = y.cpu().numpy()[rows]
    assert np.linalg.norm(yg[:N] - yr[:N]) <= 1e-12 * np.linalg.norm(yr[:N])
    assert np.linalg.norm(yg[N:] - yr[N:]) <= 1e-12 * np.linalg.norm(yr[N:])
    assert np.linalg.norm(x.cpu().numpy() - xr) <= 1e-12 * np.linalg.norm(xr)
