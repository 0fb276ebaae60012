"""Evaluation at points that no subdomain of a level covers: on an L-shaped domain, whose windows are
normalised over the kept subdomains, the value is NaN (0/0); on a box it is that of the other levels.
Covered points among them against the oracle, at the 1e-12 of the other evaluation tests."""
import dataclasses

import numpy as np
import pytest

from inputs import configs, feature_params
from oracle import evaluate as ev
from oracle import geometry as geo

from gpu_util import dev, torch_mod

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [5, 64, 70])
@pytest.mark.parametrize("domain", ["l_shape", "box"])
def test_points_off_the_supports(domain, K):
    from paper_2409_01949_amd import Problem
    torch = torch_mod()
    spec = dataclasses.replace(configs.helmholtz(omega=2.0, levels=((1, 1), (6, 6)), K=K, n=30), domain=domain)
    W, b = feature_params(spec)
    P = Problem.from_spec(spec, W, b)
    inside = np.array([[.25, .25], [.4, .9], [.02, .98], [1.2, .2], [.3, -.25]])
    off = np.array([[1.5, .2], [-.5, .5], [.2, 3.0], [3.0, 3.0], [-.3, 1.4]])
    pts = np.concatenate([off[:2], inside, off[2:]])
    coef = np.random.default_rng(K).standard_normal(P.sizes["n_phi"])
    u = torch.empty((1, len(pts)), dtype=torch.float64, device="cuda")
    P.evaluate(dev(coef), dev(pts), u)
    P.destroy()
    Wk, bk = geo.kept_parameters(spec, W, b)
    with np.errstate(invalid="ignore"):
        ref = ev.evaluate(spec, Wk, bk, coef, pts)
    got = u.cpu().numpy()[0]
    is_off = np.r_[np.ones(2, bool), np.zeros(5, bool), np.ones(3, bool)]
    if domain == "l_shape":
        assert np.all(np.isnan(got[is_off]))
    else:
        is_off[:] = False
    assert np.abs(got - ref)[~is_off].max() <= 1e-12 * np.abs(ref).max()
