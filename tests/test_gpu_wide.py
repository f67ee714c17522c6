"""The matrix kernels of 33 rows and more at the edges of their tiles.

test_products_at_tile_edges: products of single matrices (rv_debug_linear)
against float64 as the planner runs them, at row counts around its switch to
the wide kernel (33), with whole and partial token tiles.  At these sizes it
picks the 128-row shape, mostly with two token tiles (some launches with three
to six or nine), always in several token groups.  The operand is the hi/lo pair of the rows, so the
product's error is its fp32 summation: about sqrt(K) ulps of the largest
partial sum, bounded here by 4e-6 of the row's root mean square.

test_every_shape: whole passes (prefill and verify, every epilogue) with the
launch shape forced, against the oracle: 128- and 256-row workgroups of 2 - 9
token tiles, the 512-row kernel, 1 - 8 k-groups (one to 28 steps each, odd
counts among them), and row counts one below, at and one above a token tile's
edge, in one token group and in several.  A shape that does not divide a matrix
fails the call, so every matmul of 33 rows and more ran as asked.  Logits are
held to 2e-4 of the row's largest, four times the 5e-5 of the hi/lo operand
form.
"""
import numpy as np
import pytest

import oracle
import workload
from workload import ModelShape

pytestmark = pytest.mark.gpu

# d 384: QKV 1152 = 9 x 128, O 384 = 3 x 128, 12 k-steps; d 1280: 40 k-steps, down 44
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


# (width, query heads, kv heads, head dim, ffn), (rows, k-groups) to force: K of 24 and 48
# k-steps; of 56; of 16, at widths that 512 divides
FORCED = [((768, 12, 4, 64, 1536), [(r, g) for r in (128, 256) for g in (1, 2, 3, 4, 6)]),
          ((1792, 14, 2, 128, 1792), [(128, 7), (256, 7)]),
          ((512, 8, 4, 64, 512), [(128, 8), (256, 8), (512, 1)])]


@pytest.mark.parametrize("M", [33, 47, 48, 49, 143, 144, 145])
@pytest.mark.parametrize("model", FORCED, ids=lambda f: f"d{f[0][0]}")
def test_every_shape(rv, gpu, model, M):
    (d, hq, hkv, hd, F), shapes = model
    shape = ModelShape(f"forced{d}", 2, d, hq, hkv, hd, F, 1024, "bf16")
    k = 16 if M < 100 else 32  # 34 or 66 LM-head rows
    hist = [int(t) for t in workload.random_ids(shape.vocab, M + 1, 57, M)]  # M rows of prefill
    draft = workload.random_ids(shape.vocab, k, 58, M)
    probe = workload.random_ids(shape.vocab, M - 1 - 2 * k, 59, M)
    ref = oracle.verify(shape, 4, hist, draft, probe, 0.3, 0)["z"]
    limit = 2e-4 * np.abs(ref).max()
    v = rv.Verifier(shape, 4, 1, 2 * M + 8, max_block=320, max_drafts=k)
    try:
        for rows, gk in shapes:
            for mt in [8] if rows == 512 else range(2, 10):
                rv.rv_debug_force_matmul(v.cache, rows, mt, gk)
                v.prefill([hist])
                v.verify([len(hist)], draft.reshape(1, -1), probe, 0.3, 0)
                err = np.abs(v.output(rv.RV_OUT_FUSED).cpu().numpy()[0] - ref).max()
                assert err < limit, (rows, mt, gk, err, limit)
    finally:
        v.close()


def test_forced_shapes_are_checked(rv, gpu):
    shape = ModelShape("forced640", 1, 512, 8, 1, 64, 512, 512, "bf16")  # QKV 640 wide: 256 does not divide it
    v = rv.Verifier(shape, 3, 1, 128, max_block=72, max_drafts=8)
    hist = [int(t) for t in workload.random_ids(shape.vocab, 50, 60)]
    try:
        for rows, mt, gk in [(64, 4, 1), (128, 1, 1), (256, 10, 1), (128, 4, 0), (128, 4, 9), (512, 8, 2)]:
            with pytest.raises(rv.RVError) as e:
                rv.rv_debug_force_matmul(v.cache, rows, mt, gk)
            assert e.value.name == "RV_E_ARG"
        rv.rv_debug_force_matmul(v.cache, 256, 4, 1)
        with pytest.raises(rv.RVError) as e:
            v.prefill([hist])
        assert e.value.name == "RV_E_HIP" and "qkv" in str(e.value)
        rv.rv_debug_force_matmul(v.cache, 0)
        v.prefill([hist])
    finally:
        v.close()
