"""Passes of row counts around the one from which the row-wise kernels (RMSNorm,
QKV finish, attention combine) take their rows in runs per XCD, against the oracle.

With four query heads per kv head the combine's workgroups per head equal the
rows, and the prefix leaves several key splits; the counts below, at and above
the switch (24) leave whole and partial runs.  fp32 is held to 1e-4 (logits are
about 1), bf16 to 2e-4 of the row's largest, four times the 5e-5 of the hi/lo
operand form.
"""
import numpy as np
import pytest

import oracle
import workload
from workload import ModelShape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [23, 24, 25, 32, 33])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_logits(rv, gpu, dtype, rows):
    shape = ModelShape(f"rows-{dtype}", 2, 256, 8, 2, 32, 384, 512, dtype)
    k, P = 2, 4
    hist = [int(t) for t in workload.random_ids(shape.vocab, 300, 87)]
    draft = workload.random_ids(shape.vocab, k, 88)
    probe = workload.random_ids(shape.vocab, rows - 1 - 2 * k - P, 89)
    v = rv.Verifier(shape, 6, 1, 352, max_block=40, max_drafts=k)
    try:
        v.prefill([hist])
        v.verify([len(hist)], draft.reshape(1, -1), probe, 0.3, P)
        z = v.output(rv.RV_OUT_FUSED).cpu().numpy()[0]
    finally:
        v.close()
    ref = oracle.verify(shape, 6, hist, draft, probe, 0.3, P)["z"]
    assert np.abs(z - ref).max() < (1e-4 if dtype == "f32" else 2e-4 * np.abs(ref).max())
