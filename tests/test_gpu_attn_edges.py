"""Attention kernels at the edges of their key tiles and query groups.

Whole passes of two-layer models against the oracle, with prefixes around the
64-key tile and the key split, one and several query heads per kv head, and
block sizes that leave partial 16-query tiles.  fp32 models are held to 1e-4
(their logits are about 1, so 1e-4 is far above the 1e-6 of fp32 sums and far
below a wrong mask or a lost key); bf16 models to 2e-4 of the row's largest
logit, four times the 5e-5 that the hi/lo operand form is held to at these
widths.
"""
import numpy as np
import pytest

import oracle
import workload
from workload import ModelShape

pytestmark = pytest.mark.gpu


def _shape(dtype, hq, hkv, hd):
    return ModelShape(f"{dtype}-{hq}-{hkv}-{hd}", 2, 256, hq, hkv, hd, 384, 512, dtype)


CASES = [  # dtype, query heads, kv heads, head dim, prefix lengths, k, probe, P
    ("f32", 8, 2, 32, [1, 63, 64], 2, 3, 1), ("f32", 4, 4, 64, [65, 130], 4, 8, 4), ("f32", 4, 1, 128, [200, 17], 3, 0, 0),
    ("f32", 8, 8, 32, [129, 256], 0, 0, 0),
    ("bf16", 8, 2, 32, [1, 63, 64, 65], 0, 0, 0), ("bf16", 4, 1, 64, [127, 128, 129, 700], 0, 0, 0),
    ("bf16", 8, 1, 128, [511, 512, 513, 1030], 0, 0, 0), ("bf16", 4, 2, 128, [31, 33, 257], 1, 1, 0),
    ("bf16", 4, 4, 32, [300, 5], 7, 0, 0), ("bf16", 8, 2, 64, [90, 600], 5, 16, 4),
]

# Decode steps of 256 workgroups and more, which take the few-query kernel's
# nontemporal loads: 32 short sequences x 8 kv heads (256, one key split), and
# 16 with one long one (640, 1024 and 1280 with 5, 8 and 10 splits, most of them
# empty for the short sequences).
SHORT = [63, 64, 65] + [1 + b * 29 % 131 for b in range(3, 32)]
CASES += [("bf16", hq, 8, hd, lens, 0, 0, 0) for hq, hd, longest in ((16, 32, 1800), (16, 64, 1000), (8, 128, 520))
          for lens in (SHORT, SHORT[:5] + [longest] + SHORT[6:16])]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}-{c[1]}x{c[2]}x{c[3]}-{c[4][-1]}-k{c[5]}")
def test_logits_at_tile_edges(rv, gpu, case):
    dtype, hq, hkv, hd, lens, k, n_probe, P = case
    shape = _shape(dtype, hq, hkv, hd)
    lens = [max(n, P) for n in lens]
    hists = [[int(t) for t in workload.random_ids(shape.vocab, n, 77, n, b)] for b, n in enumerate(lens)]
    drafts = np.stack([workload.random_ids(shape.vocab, k, 78, b) for b in range(len(lens))]) if k else \
        np.zeros((len(lens), 0), dtype=np.int32)
    probe = workload.random_ids(shape.vocab, n_probe, 79)
    S = 1 + 2 * k + n_probe + P
    v = rv.Verifier(shape, 6, len(lens), max(lens) + S + 8, max_block=max(S, 8), max_drafts=max(k, 1))
    try:
        v.prefill(hists)
        v.verify(lens, drafts, probe, 0.3, P)
        z = v.output(rv.RV_OUT_FUSED).cpu().numpy()
    finally:
        v.close()
    for b in range(len(lens)) if len(lens) <= 8 else sorted({0, 1, 2, 5, 9, 15, len(lens) - 1}):
        ref = oracle.verify(shape, 6, hists[b], drafts[b], probe, 0.3, P)["z"]
        err = np.abs(z[b] - ref).max()
        assert err < (1e-4 if dtype == "f32" else 2e-4 * np.abs(ref).max()), (shape.name, b, err)
