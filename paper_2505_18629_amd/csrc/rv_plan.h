// Host-side planning of a pass: workspace row capacities, prefill chunks,
// matmul launch shapes and the attention key split.  Plain arithmetic with no
// HIP types, so the same code also builds for the CPU alone (the host checks
// under tests/).
#pragma once
#include <algorithm>
#include <cmath>
#include <cstddef>

enum { RV_MAX_SEGS = 128 };   // query segments of one prefill chunk

constexpr int kPrefillRows = 2048;    // rows per prefill chunk
constexpr int kMaxSplitK = 16;        // k-groups of a split matmul
constexpr int kPartBlocks = 4;        // k-groups of a whole verify block's rows that the partial buffer holds
constexpr int kSplitRows = 64;        // the few-row kernel splits K for at most this many rows
constexpr int kSplitsPerQuery = 8;    // attention partial-buffer depth per query row
constexpr int kMaxKeySplits = 64;     // key splits the combine kernel merges per query

inline int plan_round_up(int x, int a) { return (x + a - 1) / a * a; }

// Rows of the cache workspace: a verify block of every sequence, or a prefill chunk.
inline int cache_rows_cap(int batch, int max_block) {
  return plan_round_up(std::max(batch * max_block, kPrefillRows), 64);
}

// Entries (query rows x heads x splits) of the attention partial buffers.
inline size_t cache_part_entries(int rows_cap, int n_heads) {
  return (size_t)rows_cap * n_heads * kSplitsPerQuery;
}

// Rows of the matmuls' partial buffer: k-groups x rows of a split launch stay within it.
inline int cache_part_rows(int batch, int max_block) {
  return std::max(kMaxSplitK * kSplitRows, kPartBlocks * plan_round_up(batch * max_block, 64));
}

// One prefill chunk: up to rows_cap rows over (sequence, position < L - 1),
// as up to RV_MAX_SEGS segments.  Segment i is sequence sb[i], positions
// spos0[i] .. spos0[i] + sn[i] - 1, at rows srow0[i] ..; kmax is the largest
// position + 1 and max_n the longest segment.
struct PrefillChunk {
  int nseg, rows, max_n, kmax;
  int sb[RV_MAX_SEGS], spos0[RV_MAX_SEGS], sn[RV_MAX_SEGS], srow0[RV_MAX_SEGS];
};

// Fills the next chunk starting at (sequence b, position pos) and advances
// them; false when every sequence's positions 0 .. L_b - 2 are covered.
inline bool next_prefill_chunk(const int* L, int B, int rows_cap, int& b, int& pos, PrefillChunk& ch) {
  while (b < B && pos >= L[b] - 1) {
    ++b;
    pos = 0;
  }
  if (b >= B) return false;
  ch.rows = ch.nseg = ch.max_n = ch.kmax = 0;
  while (b < B && ch.rows < rows_cap && ch.nseg < RV_MAX_SEGS) {
    const int avail = L[b] - 1 - pos;
    if (avail <= 0) {
      ++b;
      pos = 0;
      continue;
    }
    const int n = std::min(avail, rows_cap - ch.rows);
    ch.sb[ch.nseg] = b;
    ch.spos0[ch.nseg] = pos;
    ch.sn[ch.nseg] = n;
    ch.srow0[ch.nseg] = ch.rows;
    ++ch.nseg;
    ch.rows += n;
    pos += n;
    ch.max_n = std::max(ch.max_n, n);
    ch.kmax = std::max(ch.kmax, pos);
  }
  return true;
}

// Queries per workgroup of the bf16 attention kernel: 128 (8 waves of one
// 16-query tile), or 192 (12 waves) where groups of 192 cover a kv head's queries
// with no more query slots.  A tile's copy then serves half as many queries
// again and three waves per SIMD hide more latency: 129-192 queries take one
// group instead of a second, mostly idle one of 128 (148 queries, the 8B shape
// with up to 8 drafts: 44 -> 35 us per launch), 360 queries (70B, 45 rows) two
// groups instead of three (320 -> 280).  With more slots it loses (215 queries,
// 14B: 36 -> 43 us).
inline int plan_attn_queries(bool bf16, int qmax) {
  return bf16 && qmax > 128 && (qmax + 191) / 192 * 192 <= (qmax + 127) / 128 * 128 ? 192 : 128;
}

inline bool plan_split_fits(int ns, int groups, int qmax, size_t part_entries) {
  return ns == 1 || (ns <= kMaxKeySplits && (size_t)ns * groups * qmax <= part_entries);
}

// Key split of one attention launch (a multiple of 64 keys).  Minimises the
// estimated time: rounds of 256 workgroups (one per CU) x (64-key tiles per
// workgroup + a per-workgroup overhead of about two tiles; 70B batch 8 with 8K
// keys: 4 splits, 768 workgroups, 348 us when this was chosen, 393 with 3 splits
// and 576) x 2.9 us per tile, counting the workgroups that have keys (segment s
// has keys 0 .. seg_end[s]-1 and G * seg_rows[s] queries per kv head, in groups
// of qpw), and for several splits the combine kernel (4 us, and 512 bytes per
// partial and output row at 3.5 TB/s; one split needs none: 2048-row prefill
// chunks otherwise split in two, 8B prefill 13.46 -> 13.94 ms).  Tile time and
// partial bytes are those of bf16 at head_dim 128; at 64 both are about half, so
// there only the 4 us weigh too little.  Several splits are bounded by the
// partial buffer (splits x segments x kv heads x qmax entries) and by the combine
// kernel's kMaxKeySplits splits per query; one split writes no partials and so
// always fits (a chunk of one long and many short prefixes can have more entries
// than the buffer, which follows its rows).
inline int plan_attn_split(int kmax, int nseg, const int* seg_end, const int* seg_rows, int n_kv, int G, int qmax,
                           size_t part_entries, int qpw = 128) {
  const int groups = nseg * n_kv;
  int ks = 0;
  double best = 0;
  for (int cand = 64; cand <= plan_round_up(kmax, 64); cand += 64) {
    const int ns = (kmax + cand - 1) / cand;
    if (!plan_split_fits(ns, groups, qmax, part_entries)) continue;
    long long wgs = 0;
    for (int s = 0; s < nseg; ++s)
      wgs += (long long)((seg_end[s] + cand - 1) / cand) * n_kv * ((G * seg_rows[s] + qpw - 1) / qpw);
    const double combine = ns > 1 ? 4 + (double)(ns + 1) * groups * qmax * 512 / 3.5e6 : 0;
    const double t = (double)((wgs + 255) / 256) * (cand / 64 + 2) * 2.9 + combine;
    if (ks == 0 || t < best) {
      best = t;
      ks = cand;
    }
  }
  return ks;
}

// At most this many queries per (segment, kv head): k_attn_few, whose waves
// share the queries and split the keys (bf16).
constexpr int kFewQueries = 16;

// Key split of one k_attn_few launch (a multiple of 64 keys; one split: no
// combine kernel; bounds as above).  Estimated us: 2.5 of launch and latency,
// the keys of a workgroup at what one CU draws (kv_bytes per key), all keys
// at what HBM gives, and for several splits the combine kernel.
inline int plan_attn_few_split(int kmax, int nseg, const int* seg_end, int n_kv, int kv_bytes, int qmax,
                               size_t part_entries) {
  const int groups = nseg * n_kv;
  long long keys = 0;
  for (int s = 0; s < nseg; ++s) keys += seg_end[s];
  const double stream = (double)keys * n_kv * kv_bytes / 5.5e6;
  int ks = 0;
  double best = 0;
  for (int cand = 64; cand <= plan_round_up(kmax, 64); cand += 64) {
    const int ns = (kmax + cand - 1) / cand;
    if (!plan_split_fits(ns, groups, qmax, part_entries)) continue;
    long long wgs = 0;
    for (int s = 0; s < nseg; ++s) wgs += (long long)((seg_end[s] + cand - 1) / cand) * n_kv;
    const double cu = (double)((wgs + 255) / 256) * std::min(cand, kmax) * kv_bytes / 4.5e4;
    const double t = 2.5 + std::max(cu, stream) + (ns > 1 ? 3.5 + 0.05 * ns : 0.0);
    if (ks == 0 || t < best) {
      best = t;
      ks = cand;
    }
  }
  return ks;
}

// Launch of one layer's attention: queries per workgroup (kFewQueries:
// k_attn_few), keys per split (a multiple of 64) and splits.
struct AttnPlan {
  int qpw, n_qgroups, ks, nsplit;
};

inline AttnPlan plan_attention(bool bf16, int kmax, int nseg, const int* seg_end, const int* seg_rows, int max_seg_rows,
                               int n_kv, int G, int hd, size_t part_entries) {
  AttnPlan p{};
  const int qmax = G * max_seg_rows;
  if (bf16 && qmax <= kFewQueries) {
    p.qpw = kFewQueries;
    p.ks = plan_attn_few_split(kmax, nseg, seg_end, n_kv, 8 * hd, qmax, part_entries);  // K and V, hi and lo planes
  } else {
    p.qpw = plan_attn_queries(bf16, qmax);
    p.ks = plan_attn_split(kmax, nseg, seg_end, seg_rows, n_kv, G, qmax, part_entries, p.qpw);
  }
  p.n_qgroups = (qmax + p.qpw - 1) / p.qpw;
  p.nsplit = (kmax + p.ks - 1) / p.ks;
  return p;
}

// Launch shape of a matmul on the wide kernel (k_wide.h): 256 or 128 output
// rows x mt token tiles per workgroup, n_tg token groups, gk k-groups.
struct WidePlan {
  bool use;      // false: plan_matmul has the launch
  bool rows256;
  int mt, n_tg, gk;
};

constexpr int kWideMinRows = 33;  // fewer rows: the few-row kernel

// The 512-row kernel (bf16): 512 output rows x 128 tokens per workgroup, batches of 4 k-steps.
constexpr int kTiledRows = 512, kTiledTokens = 128;
inline bool tiled_runs(int M, int N, int K) { return M > kSplitRows && N % kTiledRows == 0 && K / 32 % 4 == 0; }

// Estimated time (us) of one matmul whose workgroups own `rows` output rows x
// mt token tiles, `step` us per k-step.  Three limits overlap, combined as a
// 4-norm: the workgroups' own steps (each XCD -- 32 CUs, one workgroup per CU
// -- takes an equal share of them in whole rounds), the data (weights from HBM
// once at 6.2 TB/s, every workgroup's operand rows from L2 at 27 TB/s) and
// MFMA power (1.76 PFLOP/s of hi/lo products).  k-group partials are written
// at 3.3 and read by the consumer at 5 TB/s.  Fitted to 5600 launches: 16
// matrices (1B, 8B, 14B, 70B) and the LM heads at 20 - 2047 rows, every shape
// and k-group count; error 9% rms.  Over 4200 launches of the present kernel,
// operands freshly written before each, the shape it picks costs 1.0% more
// than the best one in the mean, 19% at worst (a 10 us launch).
inline double plan_matmul_us(double step, int rows, int mt, int M, int N, int K, int gk, double split_us) {
  const int n_tg = (M + 16 * mt - 1) / (16 * mt);
  const long long items = (long long)(N / rows) * gk * n_tg;
  const long long rounds = ((items + 7) / 8 + 31) / 32;
  const double work = 0.57 + (double)rounds * (0.71 + step * (K / 32 / gk));
  const double data = 3.5 + (double)N * K * 2 / 6.2e6 + (double)items * mt * 16 * (K / gk) * 4 / 2.7e7;
  const double power = 4.0 * n_tg * mt * 16 * N * K / 1.76e9;
  const double w2 = work * work, d2 = data * data, p2 = power * power;
  const double t = std::sqrt(std::sqrt(w2 * w2 + d2 * d2 + p2 * p2));
  return gk == 1 ? t : t + split_us + (double)gk * M * N * 4 * (1 / 3.3e6 + 1 / 5e6);
}

// bf16 matmuls of 33 rows and more: the cheapest of the wide kernel's shapes,
// or use = false where the 512-row kernel costs less (hundreds of rows that
// fill its 512 x 128 tiles) or no shape divides the matrix.  split_us: cost of
// splitting K beyond the partials' traffic (the QKV projection then needs its
// finish kernel).
inline WidePlan plan_wide(int M, int N, int K, bool allow_split, int part_rows, double split_us = 0) {
  WidePlan p{};
  if (M < kWideMinRows || N % 128) return p;
  const int ksteps = K / 32;
  double best = 0;
  for (int r = 0; r < 2; ++r) {
    const bool r256 = r == 1;
    const int rows = r256 ? 256 : 128;
    if (N % rows) continue;
    for (int mt = 2; mt <= 9; ++mt) {
      // us per k-step of a workgroup: 16 row tiles on 4 waves, or 8 on 4 x 2
      const double step = r256 ? 0.2886 + 0.0334 * mt : 0.1133 + 0.0306 * mt;
      for (int gk : {1, 2, 3, 4, 6, 7, 8}) {
        if (gk > 1 && (!allow_split || gk * M > part_rows)) break;
        if (ksteps % (2 * gk)) continue;  // steps of two k-steps
        const double t = plan_matmul_us(step, rows, mt, M, N, K, gk, split_us);
        if (!p.use || t < best) {
          best = t;
          p = WidePlan{true, r256, mt, (M + 16 * mt - 1) / (16 * mt), gk};
        }
      }
    }
  }
  // the 512-row kernel where it fills its rounds: 1 - 4% under two rounds of
  // 256 rows (8B gate/up at 1024 tokens 359 against 366 us, 70B at 2047 2555
  // against 2660)
  if (p.use && tiled_runs(M, N, K) && plan_matmul_us(1.07, kTiledRows, kTiledTokens / 16, M, N, K, 1, 0) < best)
    p.use = false;
  return p;
}

// Launch shape of one matmul that plan_wide leaves: row tiles per workgroup
// (nt), token tiles (mtt; both only of the few-row kernel), token groups and
// k-groups.  Aims for >= 384 workgroups (1.5 per CU)
// with as many rows per workgroup as possible, since every workgroup reads
// its k-range of all operand tiles; K is split across workgroups only for
// residual-stream outputs of few-row passes (the next RMSNorm adds the
// partials).
struct GemmPlan {
  bool tiled;  // 512-row kernel (launch_gemm_tiled)
  int nt, mtt, n_tg, gk;
};

// The matmuls plan_wide leaves: up to 32 rows, fp32, widths that 128 does not
// divide (a vocabulary of any multiple of 16), and the large ones of the
// 512-row kernel.
// part_rows: capacity of the partial buffer in rows (gk * M must fit);
// bf16: the element type (k-steps of 32, else 16); swiglu: gate/up tile pairs.
inline GemmPlan plan_matmul(bool bf16, bool swiglu, int M, int N, int K, bool allow_split, int part_rows) {
  constexpr int kTarget = 384;
  const int ksteps = K / (bf16 ? 32 : 16);
  GemmPlan p{};
  p.gk = 1;
  if (bf16 && tiled_runs(M, N, K)) {
    p.tiled = true;
    p.n_tg = (M + kTiledTokens - 1) / kTiledTokens;
    return p;
  }
  p.mtt = M <= 16 ? 1 : M <= 32 ? 2 : 4;
  p.n_tg = (M + 16 * p.mtt - 1) / (16 * p.mtt);
  const int nt_min = swiglu ? 2 : 1;
  // Large bf16 matrices against two token tiles stream best with 8 row
  // tiles per workgroup: half the operand re-reads per weight byte, and
  // ~200 workgroups already saturate HBM (8B gate/up: 5.1 -> 6.0 TB/s).
  const bool wide = bf16 && p.mtt == 2 && (long long)N * K >= (32LL << 20) && N % 128 == 0;
  if (allow_split && M <= kSplitRows && N % 64 == 0) {
    // Prefer a launch of exactly one workgroup per CU (measured at the 8B
    // shapes: down 8 tiles x 8 k-groups 22.6 -> 21.4 us, QKV 6 x 4
    // 12.8 -> 11.1 us, O 4 x 4 8.3 -> 8.1 us), with 4 and 3 row tiles tried
    // before 6: the QKV then runs 3 tiles x 2 k-groups, half the partials
    // for the finish kernel to add (the 8B batch-1 pass 3.951 -> 3.944 ms;
    // O as 2 x 2 and down as 2 x 2 or 4 x 4 measured slower).
    const int nts[] = {8, 4, 3, 6, 2};
    const int cand1[] = {2, 4, 7, 8, 14, 16};
    for (int nt : nts) {
      if ((nt == 8 && !wide) || (nt > 4 && p.mtt > 2) || N % (16 * nt)) continue;
      for (int gk : cand1) {
        if (ksteps % (4 * gk) || gk * M > part_rows) continue;
        if ((long long)(N / (16 * nt)) * gk * p.n_tg == 256) {
          p.nt = nt;
          p.gk = gk;
          return p;
        }
      }
    }
    p.nt = wide ? 8 : 4;
    const int target = wide ? kTarget / 2 : kTarget;
    const int cand[] = {1, 2, 4, 7, 8, 14, 16};
    for (int gk : cand) {
      if (ksteps % (4 * gk) || gk * M > part_rows) continue;
      p.gk = gk;
      if ((long long)(N / (16 * p.nt)) * gk * p.n_tg >= target) break;
    }
    return p;
  }
  if (wide && (long long)(N / 128) * p.n_tg >= kTarget / 2) {
    p.nt = 8;
    return p;
  }
  p.nt = 4;
  while (p.nt > nt_min && (N % (16 * p.nt) || (long long)(N / (16 * p.nt)) * p.n_tg < kTarget)) p.nt /= 2;
  while (N % (16 * p.nt)) p.nt /= 2;
  return p;
}

// Launch shape of a matmul: the wide kernel's, else plan_matmul's.
struct MatPlan {
  WidePlan wide;
  GemmPlan gemm;
  int gk() const { return wide.use ? wide.gk : gemm.gk; }
};

inline MatPlan plan_mat(bool bf16, bool swiglu, int M, int N, int K, bool allow_split, int part_rows,
                        double split_us = 0) {
  MatPlan p{};
  if (bf16) p.wide = plan_wide(M, N, K, allow_split, part_rows, split_us);
  if (!p.wide.use) p.gemm = plan_matmul(bf16, swiglu, M, N, K, allow_split, part_rows);
  return p;
}

constexpr double kQkvSplitUs = 4.0;  // a split QKV projection's finish kernel, beside its traffic

// The QKV projection: split in k-groups, or whole where that costs no more.
inline MatPlan plan_qkv(bool bf16, int M, int N, int K, int part_rows) {
  const MatPlan p = plan_mat(bf16, false, M, N, K, true, part_rows, kQkvSplitUs);
  return p.gk() > 1 ? p : plan_mat(bf16, false, M, N, K, false, part_rows);
}
