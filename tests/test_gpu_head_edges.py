"""The fusion and accept kernels at the edges of their vocabulary chunks.

rv_fuse_accept_noalloc (2048 ids per workgroup; 16-byte loads where the
vocabulary is a multiple of 4 and the logits are 16-byte aligned, single ids
otherwise) against Algorithm 2 on numpy's fp32 fusion: the decision is exact.
Equal maxima inside a lane, a wave and a chunk and across chunks go to the
lowest id, and rows may rule ids out (-inf).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _expect(o, r, x, alpha):
    z = (np.float32(1) - np.float32(alpha)) * o + np.float32(alpha) * r
    top = z.argmax(-1)  # lowest id on ties
    n = 0
    while n < len(x) and top[n] == x[n]:
        n += 1
    return n, int(top[n])


@pytest.mark.parametrize("vocab,offset", [(1, 0), (3, 0), (4, 0), (1023, 0), (2047, 0), (2048, 0), (2049, 0), (2052, 0),
                                          (4100, 0), (4100, 1), (4100, 2), (128256, 0), (128257, 0)])
def test_decisions_at_chunk_edges(rv, gpu, vocab, offset):
    import torch
    B, k, alpha = 3, 4, 0.3
    g = np.random.default_rng([vocab, offset])
    logits = g.standard_normal((B, 2 * (k + 1), vocab)).astype(np.float32)
    if vocab > 1:
        logits[g.random(logits.shape) < 0.2] = -np.inf
        logits[..., 0] = np.maximum(logits[..., 0], -3)  # a finite entry in every row
    # ties: the same large value at several ids of both rows
    for b in range(B):
        for i in range(k + 1):
            for v in g.integers(0, vocab, size=3):
                logits[b, i, v] = logits[b, k + 1 + i, v] = 9.0
    want, drafts = [], np.zeros((B, k), dtype=np.int32)
    for b in range(B):
        z = (np.float32(1) - np.float32(alpha)) * logits[b, :k + 1] + np.float32(alpha) * logits[b, k + 1:]
        drafts[b] = z.argmax(-1)[:k]
        if b and vocab > 1:
            drafts[b, b] = (drafts[b, b] + 1) % vocab
        want.append(_expect(logits[b, :k + 1], logits[b, k + 1:], drafts[b], alpha))
    buf = torch.empty(logits.size + offset, device="cuda")
    d = buf[offset:].view(logits.shape)
    d.copy_(torch.from_numpy(logits))
    acc = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    nxt = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    rv.rv_fuse_accept_noalloc(d, k, torch.from_numpy(drafts).cuda(), alpha, acc, nxt)
    torch.cuda.synchronize()
    assert list(zip(acc.tolist(), nxt.tolist())) == want
