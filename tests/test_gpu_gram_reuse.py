"""Gram blocks computed again on one problem: the launch tables and captured CG loops are kept, so a
new assembly, another kind or precision, and a preconditioner between must each give what a fresh
problem gives, bit for bit (every computation is deterministic)."""
import numpy as np
import pytest

from inputs import configs

from gpu_util import build, dev, torch_mod

pytestmark = pytest.mark.gpu


def _gram(P, spec, store, which):
    torch = torch_mod()
    P.gram(store, which)
    n = len(P.copy_gram()) * spec.K * spec.K
    G = torch.empty(n, dtype=torch.float64 if store == "fp64" else torch.float32, device="cuda")
    table = P.copy_gram(G)
    return np.array([list(t) for t in table]), G.cpu().numpy()


def _cg(P, iters):
    torch = torch_mod()
    coef = torch.empty(P.sizes["n_phi"], dtype=torch.float64, device="cuda")
    info = P.solve(coef, method="normal_cg", precond=True, iter_lim=iters, btol=0.0, check_every=4)
    assert info["iters"] == iters
    return coef.cpu().numpy()


@pytest.mark.parametrize("order", [("all", "all"), ("all", "diag", "all"), ("diag", "all", "diag")])
def test_again(order):
    spec = configs.small2d()
    f = configs.forcing(spec)
    P, *_ = build(spec, store_prec="fp32")
    for step, which in enumerate(order):
        fk = dev(f * (1.0 + step))
        for store in ("fp64", "fp32", "fp64"):
            P.assemble(fk)
            got = _gram(P, spec, store, which)
            Q, *_ = build(spec, store_prec="fp32")
            Q.assemble(fk)
            ref = _gram(Q, spec, store, which)
            assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])
            assert P.precondition(1e-3) == Q.precondition(1e-3)
            if which == "all":
                for iters in (8, 3):
                    assert np.array_equal(_cg(P, iters), _cg(Q, iters))
            Q.destroy()
    P.destroy()
