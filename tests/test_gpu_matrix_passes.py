"""M v and M^T u at the edges of their launch rules, against the oracle: blocks that fill part of a
2,048-point chunk (one, two, four and all eight point groups per thread, and one point over each),
feature counts around the multiples of 8 and 16 the passes take at a time, few and many tiles.

Tolerance: a result is a sum of n products of entries that the device and the oracle each compute
to a few ulp (1e-12 of a block's largest entry is the entry test's own bound), so the products
agree to 1e-12 of the vector's norm, as in the product tests of the core cases."""
import numpy as np
import pytest

from inputs import configs
from oracle import assemble as asm
from oracle import linalg

from gpu_util import build, dev, device_blocks, torch_mod

pytestmark = pytest.mark.gpu

# (points, subdomains, features): one subdomain holds every point of its axis
CASES = [(n, 1, K) for n in (2, 255, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4097)
         for K in (1, 8, 17)] + [(300, 3, 7), (2000, 20, 64), (900, 4, 255), (60000, 40, 16)]


@pytest.mark.parametrize("n,J,K", CASES)
def test_products(n, J, K):
    torch = torch_mod()
    spec = configs.tiny1d(K=K, J=J, n=n, delta=1.9)
    P, W, b, _ = build(spec)
    blocks = asm.assemble_blocks(spec, W, b)
    rng = np.random.default_rng(n + J + K)
    v, u = rng.standard_normal(P.sizes["n_phi"]), rng.standard_normal(n)
    y = torch.empty(n, dtype=torch.float64, device="cuda")
    x = torch.empty(len(v), dtype=torch.float64, device="cuda")
    P.matvec(dev(v), y)
    P.rmatvec(dev(u), x)
    y_ref, x_ref = asm.matvec(blocks, v, n), asm.rmatvec(blocks, u, len(v))
    P.destroy()
    assert np.linalg.norm(y.cpu().numpy() - y_ref) <= 1e-12 * np.linalg.norm(y_ref)
    assert np.linalg.norm(x.cpu().numpy() - x_ref) <= 1e-12 * np.linalg.norm(x_ref)


@pytest.mark.parametrize("store", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("n,K", [(511, 9), (1030, 33), (2300, 8)])
def test_low_precision_passes(store, n, K):
    """The vector-load passes through one refinement step of two LSQR steps: the oracle's two steps
    on the device's rounded folded entries (exact values) give y, and M c = (M R^-1) y for the
    returned c = R^-1 y.  FP64 arithmetic on the same entries throughout, cond(R) about 1e2 at
    this shift, so M c agrees to 1e-11 of its norm."""
    torch = torch_mod()
    spec = configs.tiny1d(K=K, J=1, n=n, delta=1.9)
    P, W, b, f = build(spec, store_prec=store)
    P.precondition(1e-2)
    (_, lo), = device_blocks(P, K, store, folded=True)
    (_, hi), = device_blocks(P, K, "fp64", folded=True)
    coef = torch.empty(P.sizes["n_phi"], dtype=torch.float64, device="cuda")
    y = torch.empty(n, dtype=torch.float64, device="cuda")
    P.solve(coef, method="mixed_ir", precond=True, inner_iters=2, outer_lim=1, atol=0.0, btol=0.0)
    P.matvec(coef, y)
    got = y.cpu().numpy()
    P.destroy()
    ref = linalg.lsqr(lambda v: lo @ v, lambda r: lo.T @ r, asm.rhs(spec, f), K, atol=0, btol=0,
                      iter_lim=2)
    assert np.linalg.norm(got - hi @ ref.x) <= 1e-11 * np.linalg.norm(hi @ ref.x)
