"""The two forms of the batched M V pass over the narrow copies, vector units in small batches and
matrix cores in large ones, give the same bits: instances alone against the same instances beside
others that bring the batch over each line of the rule (1,024 blocks or runs; 4,096 for widths of 25 to
47; more than 4 right-hand sides below 48 columns), for every copy, look-ahead and layout.  (The
factors of 17 to 24 columns change their form above 1,024 blocks: that case has 1,024.)"""
import numpy as np
import pytest

from inputs import configs, feature_params

from gpu_util import dev, torch_mod

pytestmark = pytest.mark.gpu


def steps(specs, R, store, patch, ahead):
    """Two refinement steps of two LSQR steps each, on M and on M R^-1: the coefficients of the
    first two instances."""
    from paper_2409_01949_amd import Batch
    torch = torch_mod()
    feats = [feature_params(s) for s in specs]
    B = Batch(specs, [w for w, _ in feats], [b for _, b in feats], R, store_prec=store)
    B.assemble(dev(np.concatenate([np.stack([configs.forcing(s) * (1.0 + 0.5 * j) for j in range(R)]).ravel()
                                   for s in specs])))
    out = []
    for precond in (False, True):
        if precond:
            B.precondition(1e-2, patch=patch)
        elif store == "fp16":
            continue            # FP16 inner solves are on the folded copy alone
        B.set_shape(store, mvb_ahead=ahead)
        coef = torch.empty(R * B.sizes["n_phi"], dtype=torch.float64, device="cuda")
        B.solve(coef, method="mixed_ir", precond=precond, inner_iters=2, outer_lim=2, check_every=2,
                atol=0.0, btol=0.0)
        out.append(coef[:R * B.offsets[2][1]].cpu().numpy())
    B.destroy()
    return out


@pytest.mark.parametrize("store", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("K,n,R,patch,blocks", [(4, 2, 5, 1, 1100), (7, 64, 8, 2, 2100), (24, 300, 6, 1, 1020),
                                                (33, 65, 8, 1, 4200), (48, 257, 1, 1, 1100),
                                                (66, 130, 3, 2, 2200), (127, 513, 2, 2, 2200),
                                                (128, 700, 8, 1, 1100)])
def test_same_bits(K, n, R, patch, blocks, store):
    own = [configs.tiny1d(K=k, J=2, n=m, delta=1.9, seed=k) for k, m in ((K, n), (max(1, K - 3), n + 1))]
    rest = [configs.tiny1d(K=3, J=blocks // 2, n=blocks, delta=1.9, seed=i) for i in (1, 2)]
    for ahead in (4, 8, 16):
        alone, beside = steps(own, R, store, patch, ahead), steps(own + rest, R, store, patch, ahead)
        assert len(alone) == len(beside) == (1 if store == "fp16" else 2)
        for a, b in zip(alone, beside):
            assert np.all(np.isfinite(a)) and np.array_equal(a, b)
