"""Prefill of one long prefix among short ones, against the oracle.

A chunk's attention partials are indexed by (segment, query of the longest
segment), so a chunk of one long and many short segments has more entries than
rows: 12 x 1699 here, beyond the 8 x 2048 that the workspace keeps per head.
Such a chunk runs as one key split, which writes its output itself.  fp32 is
held to 1e-4 (logits are about 1; fp32 sums give 1e-6), bf16 to 2e-4 of the
row's largest logit, four times the 5e-5 of the hi/lo operand form.
"""
import numpy as np
import pytest

import oracle
import workload
from workload import ModelShape

pytestmark = pytest.mark.gpu

LENS = [20] * 5 + [1700] + [20] * 6


@pytest.mark.parametrize("heads", [(8, 2, 32), (4, 4, 64), (4, 1, 128)], ids=lambda h: "x".join(map(str, h)))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_logits_after_skewed_prefill(rv, gpu, dtype, heads):
    shape = ModelShape(f"skew-{dtype}", 2, 256, *heads, 384, 512, dtype)
    hists = [[int(t) for t in workload.random_ids(shape.vocab, n, 97, b)] for b, n in enumerate(LENS)]
    draft = workload.random_ids(shape.vocab, 2, 98)
    probe = workload.random_ids(shape.vocab, 3, 99)
    v = rv.Verifier(shape, 6, len(LENS), 1720, max_block=16, max_drafts=2)
    try:
        v.prefill(hists)
        v.verify(LENS, np.stack([draft] * len(LENS)), probe, 0.3, 4)
        z = v.output(rv.RV_OUT_FUSED).cpu().numpy()
    finally:
        v.close()
    for b in (0, 5, 6, 11):
        ref = oracle.verify(shape, 6, hists[b], draft, probe, 0.3, 4)["z"]
        err = np.abs(z[b] - ref).max()
        assert err < (1e-4 if dtype == "f32" else 2e-4 * np.abs(ref).max()), (b, err)
