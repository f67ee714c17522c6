"""The matrix kernels of 33 rows and more at the edges of their tiles.

Products of single matrices (rv_debug_linear) against float64 at row counts
around the planner's switch to the wide kernel (33), whole and partial token
tiles, one and several token groups, and widths that only 128-row, only
128/256-row or also 512-row workgroups divide; reductions of few and of odd
numbers of steps.  The operand is the hi/lo pair of the rows, so the product's
error is its fp32 summation: about sqrt(K) ulps of the largest partial sum,
bounded here by 4e-6 of the row's root mean square.
"""
import numpy as np
import pytest

import oracle
from workload import ModelShape

pytestmark = pytest.mark.gpu

# d 384: QKV 1152 = 9 x 128, O 384 = 3 x 128 (128-row workgroups only), 12 k-steps;
# d 1280: O 1280 = 5 x 256, down 44 k-steps; vocab 1536 = 3 x 512
SHAPES = [ModelShape("w384", 1, 384, 12, 12, 32, 640, 1536, "bf16"),
          ModelShape("w1280", 1, 1280, 10, 10, 128, 1408, 1536, "bf16")]
ROWS = [32, 33, 47, 64, 65, 96, 113, 144, 145, 203, 289, 512, 600, 1030]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
def test_products_at_tile_edges(rv, gpu, shape):
    import torch
    v = rv.Verifier(shape, 3, 16, 128, max_block=72, max_drafts=8)
    d, F, qd = shape.d_model, shape.ffn_dim, shape.n_heads * shape.head_dim
    names = {rv.RV_MAT_QKV: ("q", "k", "v"), rv.RV_MAT_O: ("o",), rv.RV_MAT_GATEUP: ("gate", "up"),
             rv.RV_MAT_DOWN: ("down",)}
    try:
        for mat, parts in names.items():
            W = np.concatenate([oracle.weight(shape, 3, 0, n) for n in parts])
            K = {rv.RV_MAT_O: qd, rv.RV_MAT_DOWN: F}.get(mat, d)
            assert W.shape[1] == K
            for M in ROWS:
                x = np.random.default_rng([M, mat]).standard_normal((M, K)).astype(np.float32)
                hi = torch.from_numpy(x).to(torch.bfloat16)
                lo = (torch.from_numpy(x) - hi.float()).to(torch.bfloat16)
                y = torch.full((M, W.shape[0]), float("nan"), device="cuda")
                rv.rv_debug_linear(v.cache, 0, mat, torch.stack([hi, lo]).cuda().contiguous(), y)
                want = (hi.double() + lo.double()).numpy() @ W.T
                err = np.abs(y.cpu().numpy() - want).max() / np.sqrt((want ** 2).mean())
                assert err < 4e-6, (shape.name, parts, M, err)
    finally:
        v.close()
