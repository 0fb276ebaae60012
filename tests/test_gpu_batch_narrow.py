"""The batched M V pass over the narrow copies at the edges of its tiles (64 points in fours, steps of
4 features, 1 to 32 steps ahead of the block's end), one to eight right-hand sides, per subdomain
and in the patch layout's runs of 256 points, for every look-ahead.

One refinement step of two LSQR steps per right-hand side: the oracle's two steps on the device's
rounded folded entries (exact values) give y, and M c = (M R^-1) y for the returned c = R^-1 y.
FP64 arithmetic on the same entries throughout, cond(R) about 1e2 at this shift, so M c agrees to
1e-11 of its norm, as for single problems."""
import numpy as np
import pytest

from inputs import configs, feature_params
from oracle import assemble as asm
from oracle import linalg

from gpu_util import dev, torch_mod

pytestmark = pytest.mark.gpu


def _folded(B, store):
    torch = torch_mod()
    dt = {"fp64": torch.float64, "fp32": torch.float32, "bf16": torch.bfloat16,
          "fp16": torch.float16}[store]
    buf = torch.empty(B.sizes["nnz"], dtype=dt, device="cuda")
    table = B.copy_blocks(buf, store, folded=True)
    host = buf.double().cpu().numpy()
    out = []
    for row in table:
        _, _, _, nx, _, ny, K, off = (int(v) for v in row)
        out.append(host[off:off + K * nx * ny].reshape(K, nx * ny).T)
    return out


@pytest.mark.parametrize("store", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("K,n,R,patch", [(4, 2, 1, 1), (5, 63, 3, 1), (7, 64, 8, 1), (30, 65, 8, 2),
                                         (64, 257, 5, 1), (66, 300, 8, 2), (127, 513, 2, 2),
                                         (128, 700, 8, 1)])
def test_two_steps(K, n, R, patch, store):
    from paper_2409_01949_amd import Batch
    torch = torch_mod()
    specs = [configs.tiny1d(K=k, J=1, n=m, delta=1.9, seed=k) for k, m in ((K, n), (K - 3, n + 1))]
    feats = [feature_params(s) for s in specs]
    B = Batch(specs, [w for w, _ in feats], [b for _, b in feats], R, store_prec=store)
    fs = [np.stack([configs.forcing(s) * (1.0 + 0.5 * j) + j * np.arange(s.n_points[0])
                    for j in range(R)]) for s in specs]
    B.assemble(dev(np.concatenate([f.ravel() for f in fs])))
    B.precondition(1e-2, patch=patch)
    hi, lo = _folded(B, "fp64"), _folded(B, store)
    coef = torch.empty(R * B.sizes["n_phi"], dtype=torch.float64, device="cuda")
    y = torch.empty(R * B.sizes["n_rows"], dtype=torch.float64, device="cuda")
    got = []
    for ahead in (4, 8, 16):
        B.set_shape(store, rmvb_tile=32, mvb_ahead=ahead, gather_rows=1)
        B.solve(coef, method="mixed_ir", precond=True, inner_iters=2, outer_lim=1, check_every=2,
                atol=0.0, btol=0.0)
        B.matvec(coef, y)
        got.append(y.cpu().numpy())
    B.destroy()
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])
    r0 = 0
    for s, f, H, L in zip(specs, fs, hi, lo):
        m = s.n_points[0]
        Y = got[0][R * r0:R * (r0 + m)].reshape(R, m)
        r0 += m
        for j in range(R):
            x = linalg.lsqr(lambda v: L @ v, lambda u: L.T @ u, asm.rhs(s, f[j]), L.shape[1],
                            atol=0, btol=0, iter_lim=2).x
            assert np.linalg.norm(Y[j] - H @ x) <= 1e-11 * np.linalg.norm(H @ x)
