"""The scratch of the batched block-Jacobi factors: where two matrix sets of all blocks do not fit in
free device memory the blocks go through it in chunks, with the same bits."""
import dataclasses

import pytest

from inputs import configs, feature_params

from gpu_util import dev, torch_mod

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("patch", [1, 2])
def test_little_free_memory(patch):
    from paper_2409_01949_amd import Batch
    torch = torch_mod()
    # 16,384 blocks of 128 columns: 2 GiB of Gram blocks (over patches of 2 x 2, 8 GiB)
    spec = dataclasses.replace(configs.small2d(), n_points=(160, 160), levels=((128, 128),), K=128)
    W, b = feature_params(spec)
    B = Batch([spec], [W], [b], 1)
    B.assemble(dev(configs.forcing(spec)))
    coef = [torch.empty(B.sizes["n_phi"], dtype=torch.float64, device="cuda") for _ in range(2)]
    hold = None
    try:
        for c in coef:
            B.precondition(1e-3, patch=patch)
            B.solve(c, iter_lim=3, atol=0.0, btol=0.0, check_every=3, precond=True)
            torch.cuda.synchronize()
            if hold is None:   # leave room for one matrix set, not for two
                torch.cuda.empty_cache()
                free = torch.cuda.mem_get_info()[0]
                hold = torch.empty(free - (2400 << 20), dtype=torch.uint8, device="cuda")
        assert torch.equal(coef[0], coef[1])
    finally:
        B.destroy()
        del hold
        torch.cuda.empty_cache()
