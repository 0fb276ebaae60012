"""How many products a Gram accumulator sums before a partial is written: at most 4,096 points.

One subdomain a level, zero weights and the identity operator make every stored entry the same
constant c, so a block is N c^2 and its error that of the sums alone.  A sum of n equal products in
one chain, each addition rounded to nearest, is off by at most n 0.375 2^-24 of itself (with x in
[1, 2) the final sum over its power of two, the additions in that binade are n (x - 1)/x and round
by at most the sum's 2^-24/x, those below add n/(3 x^2): (x - 2/3)/x^2 <= 0.375): 9.2e-5 at 4,096
points.  The partials of the N / 4096 = 121 chunks add at most 121 2^-25 = 3.6e-6.  The bias is one
whose chain of 8,192 is off by 1.2e-4."""
import dataclasses

import numpy as np
import pytest

from inputs import configs

from gpu_util import dev, torch_mod

pytestmark = pytest.mark.gpu


def test_fp32_chain():
    from paper_2409_01949_amd import Problem
    torch = torch_mod()
    n, levels = 704, 8     # 36 pairs of 495,616 points: enough that only the cap bounds the chunks
    spec = dataclasses.replace(configs.small2d(), n_points=(n, n), K=1, levels=((1, 1),) * levels,
                               op="identity", ansatz="none")
    P = Problem.from_spec(spec, np.zeros((levels, 2)), np.full(levels, 0.83099), "fp32")
    P.assemble(dev(np.zeros(n * n)))
    M = torch.empty(P.sizes["nnz"], dtype=torch.float32, device="cuda")
    P.copy_blocks(M, prec="fp32")
    G = torch.empty(P.sizes["n_pairs"], dtype=torch.float32, device="cuda")
    P.gram("fp32", "all")
    P.copy_gram(G)
    P.destroy()
    c = float(M[0])
    assert bool((M == c).all())
    err = np.abs(G.double().cpu().numpy() / (n * n * c * c) - 1.0).max()
    assert err <= 4096 * 0.375 * 2.0 ** -24 + 121 * 2.0 ** -25
