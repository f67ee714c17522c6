"""The work that users of this framework have it do, as cases to time.

A case is one call (or one call and the read-back of its results) through the
public entry points, on a model whose weights, cache and prefilled prefixes
the program already holds:

  verify    rv_verify / rv_verify_ragged / rv_verify_sampled: one reflective
            verification pass of the target model, and, with k = 0 and no
            probe, one plain decode step (what a draft model runs k times per
            round); the fused logits and log-probabilities are read back.
  prefill   rv_prefill_cache over new prompts and the decode step that scores
            their last token (time to first token); the logits and the last
            layer's K and V are read back.
  decide    rv_fuse_accept_noalloc: the decision alone, on logits the caller
            has.

The model shapes are those of `workload`; the larger ones run with a few of
their (identical) layers, so that several states fit on the card and a state
is quick to make.  One case is the whole 32-layer 8B pass.
"""
import math

import numpy as np
import torch

import paper_2505_18629_amd as rv
import workload

SHAPES = {
    "tiny": workload.TINY,                  # fp32
    "tiny-gqa": workload.TINY_GQA_BF16,
    "1b": workload.LLAMA1B,
    "8b": workload.LLAMA8B,
    "14b": workload.QWEN14B,
    "70b": workload.LLAMA70B,
}
RULES = {"greedy": rv.RV_RULE_GREEDY, "typical": rv.RV_RULE_TYPICAL, "sampling": rv.RV_RULE_SAMPLING}


def _verify(name, shape, layers, batch, lo, hi, k, probe, P, rule="greedy", ragged=False, alpha=0.3, temperature=1.0):
    return {"name": name, "kind": "verify", "shape": shape, "layers": layers, "batch": batch, "len_lo": lo,
            "len_hi": hi, "k": k, "probe": probe, "P": P, "rule": rule, "ragged": ragged, "alpha": alpha,
            "temperature": temperature}


def _prefill(name, shape, layers, batch, lo, hi):
    return {"name": name, "kind": "prefill", "shape": shape, "layers": layers, "batch": batch, "len_lo": lo,
            "len_hi": hi}


def _decide(name, batch, k, vocab, rule="greedy", alpha=0.3):
    return {"name": name, "kind": "decide", "batch": batch, "k": k, "vocab": vocab, "rule": rule, "alpha": alpha}


def listed():
    return [
        # the fp32 configuration's verify pass: the smallest model, all launch latency
        _verify("verify-tiny-f32", "tiny", 2, 1, 128, 128, 4, 8, 4),
        # one draft-model decode step for one user: k of these per speculative round
        _verify("decode-1b", "1b", 16, 1, 1024, 1024, 0, 0, 0, alpha=0.0),
        # the same step for a batch of users with unlike context lengths
        _verify("decode-1b-b16", "1b", 16, 16, 300, 1900, 0, 0, 0, alpha=0.0),
        # the benchmark's pass: whole 8B model, one user, Table 5's settings
        _verify("verify-8b", "8b", 32, 1, 1024, 1024, 5, 16, 4),
        # a serving batch of verify passes with unlike context lengths
        _verify("verify-8b-b16", "8b", 8, 16, 512, 4096, 5, 16, 4),
        # a draft count per sequence, entropy-thresholded acceptance
        _verify("verify-8b-dynamic", "8b", 8, 7, 333, 1501, 8, 16, 4, rule="typical", ragged=True),
        # speculative sampling at the paper's temperature, a small batch
        _verify("verify-8b-sampled", "8b", 8, 3, 700, 900, 5, 16, 4, rule="sampling", temperature=0.8),
        # the 14B shape's small batch
        _verify("verify-14b-b4", "14b", 8, 4, 2048, 2048, 7, 24, 4),
        # the 70B shape's batch on long contexts: the largest pass
        _verify("verify-70b-b8", "70b", 3, 8, 8192, 8192, 8, 24, 4),
        # a long prompt for the target model
        _prefill("prefill-8b", "8b", 4, 1, 4001, 4001),
        # several short prompts for the draft model
        _prefill("prefill-1b-short", "1b", 16, 4, 60, 300),
        # the decision alone, on logits from elsewhere
        _decide("decide-b4", 4, 5, 128256),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["verify", "verify", "verify", "decode", "decode", "prefill", "decide"])
    if kind == "decide":
        return _nameless(_decide("", _log_int(rng, 1, 16), rng.randint(0, 8), rng.choice([4096, 32000, 128256, 152064]),
                                 rng.choice(["greedy", "typical"]), rng.choice([0.0, 0.3, 0.7])))
    shape = rng.choice(["tiny", "tiny-gqa", "1b", "8b", "8b", "14b", "70b"])
    layers = {"tiny": 2, "tiny-gqa": 2, "1b": rng.choice([8, 16]), "8b": rng.choice([2, 8]), "14b": rng.choice([2, 6]),
              "70b": rng.choice([1, 2])}[shape]
    if kind == "prefill":
        batch = _log_int(rng, 1, 8)
        hi = _log_int(rng, 17, {"70b": 2000, "14b": 3000, "tiny": 1000}.get(shape, 4000) // batch)
        return _nameless(_prefill("", shape, layers, batch, rng.randint(max(2, hi // 3), hi), hi))
    batch = _log_int(rng, 1, 16)
    most = {"tiny": 1024, "tiny-gqa": 2048, "70b": 40000 // batch, "14b": 24000 // batch}.get(shape, 32000 // batch)
    hi = _log_int(rng, 40, min(8192, most))
    lo = rng.randint(max(24, hi // 4), hi)
    if kind == "decode":
        return _nameless(_verify("", shape, layers, batch, lo, hi, 0, 0, 0, alpha=0.0))
    rule = rng.choice(["greedy", "greedy", "typical", "sampling"])
    k = rng.randint(1, 9)
    return _nameless(_verify("", shape, layers, batch, lo, hi, k, rng.randint(0, 28), rng.randint(0, 8), rule,
                             rule != "sampling" and rng.random() < 0.3, rng.choice([0.0, 0.3, 0.6]),
                             0.8 if rule == "sampling" else 1.0))


def _nameless(case):
    del case["name"]
    return case


# ------------------------------------------------------------------ sizes

def _shape(case):
    return SHAPES[case["shape"]].with_layers(case["layers"])


def _spread(lo, hi, n):
    """n values from hi down to lo, in a mixed order."""
    return [hi if n == 1 else lo + (hi - lo) * ((5 * b + 1) % n if n % 5 else b) // (n - 1) for b in range(n)]


def _lens(case):
    return _spread(case["len_lo"], case["len_hi"], case["batch"])


def _draft_counts(case):
    return _spread(0, case["k"], case["batch"]) if case["ragged"] else [case["k"]] * case["batch"]


# ----------------------------------------------------------------- inputs

def _ids(case, seed):
    """Prefix ids [batch][longest], draft ids [batch][max(k, 1)] and probe ids, on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    V = _shape(case).vocab

    def draw_ids(*dims):
        return torch.randint(0, V, dims, generator=g, device="cuda", dtype=torch.int32)

    return draw_ids(case["batch"], case["len_hi"]), draw_ids(case["batch"], max(case.get("k", 0), 1)), \
        draw_ids(max(case.get("probe", 0), 1))


def _draft_probs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed + (1 << 20))
    V = _shape(case).vocab
    q = torch.randn((case["batch"], case["k"], V), generator=g, device="cuda")
    return torch.softmax(q, -1).contiguous()


def _decide_inputs(case, seed):
    """Logits of the spread a language model's have; about 70% of the drafts are the fused argmax."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, k, V = case["batch"], case["k"], case["vocab"]
    logits = torch.randn((B, 2 * (k + 1), V), generator=g, device="cuda") * 2.5
    fused = (1 - case["alpha"]) * logits[:, :k] + case["alpha"] * logits[:, k + 1:2 * k + 1]
    other = torch.randint(0, V, (B, k), generator=g, device="cuda")
    keep = torch.rand((B, k), generator=g, device="cuda") < 0.7
    return logits, torch.where(keep, fused.argmax(-1), other).to(torch.int32).contiguous()


def prepare(case, seed):
    if case["kind"] == "decide":
        logits, drafts = _decide_inputs(case, seed)
        out = torch.zeros((2, case["batch"]), dtype=torch.int32, device="cuda")
        return {"case": case, "logits": logits, "drafts": drafts, "accept_len": out[0], "next_id": out[1]}
    shape, lens = _shape(case), _lens(case)
    ids, drafts, probe = _ids(case, seed)
    S = 1 + 2 * case.get("k", 0) + case.get("probe", 0) + case.get("P", 0)
    v = rv.Verifier(shape, seed % 1000, case["batch"], case["len_hi"] + S + 8, max_block=max(S, 8),
                    max_drafts=max(case.get("k", 0), 4))
    st = {"case": case, "v": v, "lens": np.asarray(lens, dtype=np.int32), "ids": ids, "drafts": drafts, "probe": probe}
    if case["kind"] == "verify":
        rv.rv_prefill_cache(v.cache, ids, lens)
        st["kb"] = _draft_counts(case)
        if case["rule"] == "sampling":
            st["q"] = _draft_probs(case, seed)
    return st


# -------------------------------------------------------------------- run

def _decode(v, lens):
    rv.rv_verify(v.cache, lens, None, 0, None, 0, 0.0, 0, v.accept_len, v.next_id)
    v.k, v.kb = 0, None


def run(st):
    c = st["case"]
    if c["kind"] == "decide":
        rv.rv_fuse_accept_noalloc(st["logits"], c["k"], st["drafts"] if c["k"] else None, c["alpha"],
                                  st["accept_len"], st["next_id"], rule=RULES[c["rule"]])
        return {"accept_len": st["accept_len"], "next_id": st["next_id"]}
    v, lens = st["v"], st["lens"]
    if c["kind"] == "prefill":
        rv.rv_prefill_cache(v.cache, st["ids"], lens)
        _decode(v, lens)
        out = {"next_id": v.next_id, "z": v.output(rv.RV_OUT_FUSED)}
        sh = v.shape
        for b, n in enumerate(lens):
            dims = ((2,) if sh.dtype == "bf16" else ()) + (sh.n_kv_heads, int(n) - 1, sh.head_dim)
            kv = torch.empty((2,) + dims, dtype=torch.bfloat16 if sh.dtype == "bf16" else torch.float32, device="cuda")
            rv.rv_debug_export_kv(v.cache, sh.n_layers - 1, b, 0, int(n) - 1, kv[0], kv[1])
            out["kv%d" % b] = kv.float().sum(1) if sh.dtype == "bf16" else kv  # hi + lo
        return out
    k, n_probe = c["k"], c["probe"]
    probe, drafts = (st["probe"] if n_probe else None), (st["drafts"] if k else None)
    if c["rule"] == "sampling":
        rv.rv_verify_sampled(v.cache, lens, drafts, k, st["q"], probe, n_probe, c["alpha"], c["P"], 12345,
                             v.accept_len, v.next_id, temperature=c["temperature"])
    elif c["ragged"]:
        rv.rv_verify_ragged(v.cache, lens, st["drafts"], max(k, 1), st["kb"], probe, n_probe, c["alpha"], c["P"],
                            v.accept_len, v.next_id, rule=RULES[c["rule"]])
    else:
        rv.rv_verify(v.cache, lens, drafts, k, probe, n_probe, c["alpha"], c["P"], v.accept_len, v.next_id,
                     rule=RULES[c["rule"]], temperature=c["temperature"])
    v.k, v.kb = (max(k, 1) if c["ragged"] else k), (st["kb"] if c["ragged"] else None)
    return {"accept_len": v.accept_len, "next_id": v.next_id, "z": v.output(rv.RV_OUT_FUSED),
            "logp": v.output(rv.RV_OUT_LOGP_FUSED)}


# ------------------------------------------------------------- accounting

def work(case):
    """Weights read once, the cached prefix read once (hi and lo planes of a bf16 model's K and V), the new K and V
    written, the results written; two flops per multiply-add of the matrices and of attention."""
    if case["kind"] == "decide":
        n = case["batch"] * (case["k"] + 1) * case["vocab"]
        return {"bytes": 8 * n, "flops": 40 * n}
    sh, lens = _shape(case), _lens(case)
    d, qd, kvd, F, V, L = sh.d_model, sh.n_heads * sh.head_dim, sh.n_kv_heads * sh.head_dim, sh.ffn_dim, sh.vocab, sh.n_layers
    w = 2 if sh.dtype == "bf16" else 4
    layer = d * (qd + 2 * kvd) + qd * d + 3 * F * d
    if case["kind"] == "prefill":
        new, first, counts = [n for n in lens], [0] * len(lens), [0] * len(lens)
    else:
        counts = _draft_counts(case)
        new = [1 + 2 * kb + case["probe"] + case["P"] for kb in counts]
        first = [n - 1 for n in lens]
    rows, heads = sum(new), sum(2 * (kb + 1) for kb in counts)
    keys = sum(s * (p + (s + 1) / 2) for s, p in zip(new, first))
    read = L * layer * w + V * d * w + sum(first) * 2 * kvd * 4 * L + rows * d * w
    wrote = rows * 2 * kvd * 4 * L + heads // 2 * V * 4 * 2
    return {"bytes": read + wrote, "flops": 2 * layer * L * rows + 2 * V * d * heads + 4 * qd * L * keys}


def tolerance(case):
    """About four times the distance from `exact` measured over these ranges: 3e-7 (fp32), 2e-5 - 4e-5 (bf16 weights,
    hi/lo activations, up to 16 layers) and 7e-5 (32 layers) of the logits."""
    if case["kind"] == "decide":
        return "exact"
    if SHAPES[case["shape"]].dtype == "f32":
        return {"rel": 2e-6, "differ": 0.01}
    return {"rel": 1.6e-4 if case["layers"] <= 16 else 3e-4, "differ": 0.01}


# ------------------------------------------------------------------ exact

def _mix(z):
    """splitmix64's finaliser of z + golden on int64 tensors (the arithmetic wraps; shifts are made logical)."""
    z = z + (0x9E3779B97F4A7C15 - (1 << 64))
    z = (z ^ ((z >> 30) & ((1 << 34) - 1))) * (0xBF58476D1CE4E5B9 - (1 << 64))
    z = (z ^ ((z >> 27) & ((1 << 37) - 1))) * (0x94D049BB133111EB - (1 << 64))
    return z ^ ((z >> 31) & ((1 << 33) - 1))


class _Weights:
    """The seeded weights of include/rv.h's rv_init_weights, in 64 bits."""

    def __init__(self, sh, seed):
        self.sh, self.seed = sh, _mix(torch.tensor(seed, dtype=torch.int64, device="cuda"))
        self.scale = float(np.float32(sh.init_std / math.sqrt(4.0 * (65536.0 * 65536.0 - 1.0) / 12.0)))

    def at(self, t, i):
        h = _mix((i + (t << 36)) ^ self.seed)
        s = (h & 0xFFFF) + ((h >> 16) & 0xFFFF) + ((h >> 32) & 0xFFFF) + ((h >> 48) & 0xFFFF) - 2 * 65535
        w = s.to(torch.float32) * self.scale
        return (w.to(torch.bfloat16) if self.sh.dtype == "bf16" else w).to(torch.float64)

    def times(self, t, out, x):
        """x . W^T of tensor t, [rows][out]."""
        n_in = x.shape[-1]
        y = torch.empty((x.shape[0], out), dtype=torch.float64, device="cuda")
        step = max(1, (1 << 27) // n_in)
        for r in range(0, out, step):
            n = min(step, out - r)
            i = torch.arange(r * n_in, (r + n) * n_in, device="cuda", dtype=torch.int64)
            y[:, r:r + n] = x @ self.at(t, i).view(n, n_in).t()
        return y

    def rows(self, ids):
        d = self.sh.d_model
        return self.at(0, ids.to(torch.int64)[:, None] * d + torch.arange(d, device="cuda"))


def _norm(h, eps):
    return h * torch.rsqrt((h * h).mean(-1, keepdim=True) + eps)


def _rotate(x, pos, base):
    hd = x.shape[-1]
    a = pos.to(torch.float64)[:, None] * (base ** (-2.0 * torch.arange(hd // 2, device="cuda", dtype=torch.float64) / hd))
    c, s = torch.cos(a)[:, None], torch.sin(a)[:, None]
    u, w = x[..., :hd // 2], x[..., hd // 2:]
    return torch.cat([u * c - w * s, w * c + u * s], -1)


def _attend(q, k, v, pos):
    """Causal attention of one sequence: q [rows][heads][hd] at positions pos, k and v [keys][kv heads][hd]."""
    n, H, hd = q.shape
    G = H // k.shape[1]
    out = torch.empty_like(q)
    keys = torch.arange(k.shape[0], device="cuda")
    step = max(1, (1 << 27) // k.shape[0] // G)
    for g in range(k.shape[1]):
        for r in range(0, n, step):
            qq = q[r:r + step, g * G:(g + 1) * G].reshape(-1, hd)
            s = (qq @ k[:, g].t()).view(-1, G, k.shape[0]) / math.sqrt(hd)
            s.masked_fill_(keys > pos[r:r + step, None, None], -math.inf)
            out[r:r + step, g * G:(g + 1) * G] = (torch.softmax(s, -1).view(-1, k.shape[0]) @ v[:, g]).view(-1, G, hd)
    return out


def _forward(sh, seed, seqs, rows):
    """Logits of the given rows of every sequence (from scratch), and the last layer's rotated K, and V."""
    W = _Weights(sh, seed)
    hd, qd, kvd = sh.head_dim, sh.n_heads * sh.head_dim, sh.n_kv_heads * sh.head_dim
    at = np.cumsum([0] + [len(s) for s in seqs])
    pos = torch.cat([torch.arange(len(s), device="cuda") for s in seqs])
    h = W.rows(torch.cat(seqs))
    keep = torch.cat([torch.as_tensor(r, device="cuda") + int(a) for r, a in zip(rows, at)])
    for l in range(sh.n_layers):
        t, last = 1 + 7 * l, l + 1 == sh.n_layers
        x = _norm(h, sh.rms_eps)
        k = _rotate(W.times(t + 1, kvd, x).view(-1, sh.n_kv_heads, hd), pos, sh.rope_base)
        v = W.times(t + 2, kvd, x).view(-1, sh.n_kv_heads, hd)
        use = keep if last else torch.arange(len(h), device="cuda")  # past its K and V the last layer needs only these
        q = _rotate(W.times(t, qd, x[use]).view(-1, sh.n_heads, hd), pos[use], sh.rope_base)
        a = torch.empty_like(q)
        for b in range(len(seqs)):
            mine = (use >= int(at[b])) & (use < int(at[b + 1]))
            a[mine] = _attend(q[mine], k[at[b]:at[b + 1]], v[at[b]:at[b + 1]], pos[use][mine])
        h = h[use] + W.times(t + 3, sh.d_model, a.reshape(len(use), qd))
        x = _norm(h, sh.rms_eps)
        f = torch.nn.functional.silu(W.times(t + 4, sh.ffn_dim, x)) * W.times(t + 5, sh.ffn_dim, x)
        h = h + W.times(t + 6, sh.d_model, f)
    logits = W.times(1 + 7 * sh.n_layers, sh.vocab, _norm(h, sh.rms_eps))
    return logits, [(k[at[b]:at[b + 1]], v[at[b]:at[b + 1]]) for b in range(len(seqs))]


def exact(case, seed):
    if case["kind"] == "decide":
        return None  # whole numbers only
    sh, lens = _shape(case), _lens(case)
    ids, drafts, probe = _ids(case, seed)
    if case["kind"] == "prefill":
        z, kv = _forward(sh, seed % 1000, [ids[b, :n] for b, n in enumerate(lens)], [[n - 1] for n in lens])
        out = {"next_id": None, "z": z.view(len(lens), 1, -1)}
        for b, (k, v) in enumerate(kv):
            out["kv%d" % b] = torch.stack([k[:-1].transpose(0, 1), v[:-1].transpose(0, 1)])
        return out
    counts, n_probe, P = _draft_counts(case), case["probe"], case["P"]
    seqs, rows = [], []
    for b, (n, kb) in enumerate(zip(lens, counts)):
        x = drafts[b, :kb]
        seqs.append(torch.cat([ids[b, :n], x, probe[:n_probe], ids[b, n - P:n], x]))
        shift = kb + n_probe + P
        rows.append([n - 1 + i for i in range(kb + 1)] + [n - 1 + shift + i for i in range(kb + 1)])
    logits, _ = _forward(sh, seed % 1000, seqs, rows)
    z, r0 = [], 0
    for kb in counts:
        o, r = logits[r0:r0 + kb + 1], logits[r0 + kb + 1:r0 + 2 * kb + 2]
        z.append(((1 - case["alpha"]) * o + case["alpha"] * r) / case["temperature"])
        r0 += 2 * kb + 2
    z = torch.cat(z)
    if not case["ragged"]:
        z = z.view(case["batch"], case["k"] + 1, -1)
    return {"accept_len": None, "next_id": None, "z": z, "logp": torch.log_softmax(z, -1)}
