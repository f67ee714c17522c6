// CPU check of the library's host-side planning (rv_plan.h) at the shapes of
// the benchmark workloads and at edge cases: every prefill chunk stays inside
// the workspace and segment arrays and covers each sequence's positions once,
// every attention launch's key split fits the partial buffer and the grid
// limits, and every matmul launch shape is one the launchers instantiate.  The
// plans are those of plan_attention, plan_mat and plan_qkv, which the passes use.
// Built with the address and undefined-behaviour sanitizers by
// tests/test_host_checks.py; exits non-zero on the first violation.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "rv_plan.h"

namespace {

int failures = 0;
long long n_wide = 0, n_tiled = 0, n_few = 0;  // matmul plans by kernel

#define CHECK(cond, ...)                          \
  do {                                            \
    if (!(cond)) {                                \
      std::fprintf(stderr, "FAIL %s: ", #cond);   \
      std::fprintf(stderr, __VA_ARGS__);          \
      std::fprintf(stderr, "\n");                 \
      ++failures;                                 \
      return;                                     \
    }                                             \
  } while (0)

struct Shape {
  const char* name;
  int n_heads, n_kv, hd;
  bool bf16;
};

// One attention launch over segments (seg_end, seg_rows): the split, the
// partial-buffer entries and the grids of the attention and combine kernels.
void check_attention(const Shape& sh, int kmax, int nseg, const int* seg_end, const int* seg_rows, int max_seg_rows,
                     size_t part_entries, const char* what) {
  const int G = sh.n_heads / sh.n_kv;
  const int qmax = G * max_seg_rows;
  const AttnPlan p = plan_attention(sh.bf16, kmax, nseg, seg_end, seg_rows, max_seg_rows, sh.n_kv, G, sh.hd, part_entries);
  CHECK(p.qpw == 128 || (sh.bf16 && (p.qpw == 192 || (p.qpw == 16 && qmax <= 16))), "%s %s: %d queries per workgroup",
        sh.name, what, p.qpw);
  CHECK((long long)p.n_qgroups * p.qpw >= qmax && (long long)(p.n_qgroups - 1) * p.qpw < qmax, "%s %s: query groups",
        sh.name, what);
  CHECK(p.ks > 0 && p.ks % 64 == 0, "%s %s: no key split for kmax %d", sh.name, what, kmax);
  const long long nsplit = p.nsplit;
  CHECK(nsplit == (kmax + p.ks - 1) / p.ks && nsplit <= kMaxKeySplits, "%s %s: %lld splits", sh.name, what, nsplit);
  // one split writes the output and no partials
  CHECK(nsplit == 1 || (size_t)nsplit * nseg * sh.n_kv * qmax <= part_entries, "%s %s: partial entries", sh.name, what);
  const long long units = nsplit * nseg * sh.n_kv;
  const long long grid = (units + 7) / 8 * 8 * p.n_qgroups;
  CHECK(grid > 0 && grid < (1LL << 31), "%s %s: attention grid %lld", sh.name, what, grid);
  CHECK(sh.bf16 || p.n_qgroups < 65536, "%s %s: fp32 attention grid", sh.name, what);
  CHECK((long long)(qmax + 3) / 4 < (1LL << 31) && (long long)nseg * sh.n_kv < 65536, "%s %s: combine grid", sh.name,
        what);
  for (int s = 0; s < nseg; ++s) CHECK(seg_end[s] <= kmax, "%s %s: segment %d ends past kmax", sh.name, what, s);
}

// Prefill of `L` (one length per sequence) in a cache of B sequences with
// blocks of up to max_block rows.
void check_prefill(const Shape& sh, const std::vector<int>& L, int max_block, int max_len) {
  const int B = (int)L.size();
  const int rows_cap = cache_rows_cap(B, max_block);
  const size_t part = cache_part_entries(rows_cap, sh.n_heads);
  std::vector<long long> covered(B, 0);
  std::vector<int> next_pos(B, 0);
  int b = 0, pos = 0, chunks = 0;
  PrefillChunk ch;
  while (next_prefill_chunk(L.data(), B, rows_cap, b, pos, ch)) {
    ++chunks;
    CHECK(ch.nseg >= 1 && ch.nseg <= RV_MAX_SEGS, "%s: chunk %d has %d segments", sh.name, chunks, ch.nseg);
    CHECK(ch.rows >= 1 && ch.rows <= rows_cap, "%s: chunk %d has %d rows (cap %d)", sh.name, chunks, ch.rows, rows_cap);
    int row = 0, seg_end[RV_MAX_SEGS];
    for (int i = 0; i < ch.nseg; ++i) {
      const int s = ch.sb[i];
      CHECK(s >= 0 && s < B, "%s: segment sequence %d", sh.name, s);
      CHECK(ch.srow0[i] == row, "%s: segment rows not consecutive", sh.name);
      CHECK(ch.sn[i] >= 1 && ch.spos0[i] == next_pos[s] && ch.spos0[i] + ch.sn[i] <= L[s] - 1,
            "%s: segment %d of sequence %d covers %d..%d (L %d, next %d)", sh.name, i, s, ch.spos0[i],
            ch.spos0[i] + ch.sn[i] - 1, L[s], next_pos[s]);
      CHECK(ch.spos0[i] + ch.sn[i] <= max_len, "%s: position past max_len", sh.name);
      next_pos[s] += ch.sn[i];
      covered[s] += ch.sn[i];
      row += ch.sn[i];
      seg_end[i] = ch.spos0[i] + ch.sn[i];
      CHECK(ch.sn[i] <= ch.max_n && seg_end[i] <= ch.kmax, "%s: chunk extents", sh.name);
    }
    CHECK(row == ch.rows, "%s: rows", sh.name);
    check_attention(sh, ch.kmax, ch.nseg, seg_end, ch.sn, ch.max_n, part, "prefill");
    if (failures) return;
  }
  for (int s = 0; s < B; ++s)
    CHECK(covered[s] == std::max(L[s] - 1, 0), "%s: sequence %d covered %lld of %d", sh.name, s, covered[s], L[s] - 1);
  std::printf("%s prefill B=%d: %d chunks, rows_cap %d, partial entries %zu\n", sh.name, B, chunks, rows_cap, part);
}

// A verify pass: one segment of S rows per sequence at positions L-1 ...
void check_verify(const Shape& sh, const std::vector<int>& L, int S, int max_block) {
  const int B = (int)L.size();
  const int rows_cap = cache_rows_cap(B, max_block);
  CHECK(S <= max_block && B * S <= rows_cap, "%s: verify rows", sh.name);
  std::vector<int> seg_end(B), seg_rows(B, S);
  int kmax = 0;
  for (int b = 0; b < B; ++b) {
    seg_end[b] = L[b] - 1 + S;
    kmax = std::max(kmax, seg_end[b]);
  }
  check_attention(sh, kmax, B, seg_end.data(), seg_rows.data(), S, cache_part_entries(rows_cap, sh.n_heads), "verify");
  std::printf("%s verify B=%d S=%d: ok\n", sh.name, B, S);
}

// One matmul launch as planned: the shape must be one the launchers
// instantiate, divide N into whole row groups and K into whole k-step
// batches, fit the partial buffer and the grid limit.
void check_launch(const char* what, bool bf16, bool swiglu, bool allow_split, int M, int N, int K, int part_rows,
                  const MatPlan& mp) {
  const int ksteps = K / (bf16 ? 32 : 16);
  const int gk = mp.gk();
  CHECK(gk >= 1 && (gk == 1 || allow_split), "%s M=%d: k-groups %d", what, M, gk);
  CHECK(gk == 1 || (long long)gk * M <= part_rows, "%s M=%d: %d k-groups x %d rows past %d", what, M, gk, M, part_rows);
  const GemmPlan& p = mp.gemm;
  if (mp.wide.use) {
    ++n_wide;
    const WidePlan& w = mp.wide;
    const int rows = w.rows256 ? 256 : 128;
    CHECK(bf16 && M >= kWideMinRows && w.mt >= 2 && w.mt <= 9, "%s M=%d: no wide kernel of %d token tiles", what, M, w.mt);
    CHECK(N % rows == 0 && ksteps % (2 * gk) == 0, "%s M=%d: N %d, %d k-steps, %d k-groups", what, M, N, ksteps, gk);
    CHECK(gk <= 8, "%s M=%d: %d k-groups past what the consumers add", what, M, gk);
    CHECK((long long)w.n_tg * w.mt * 16 >= M && (long long)(N / rows) * gk * w.n_tg < (1LL << 30), "%s M=%d: token groups",
          what, M);
  } else if (p.tiled) {
    ++n_tiled;
    CHECK(bf16 && M >= kWideMinRows && p.gk == 1, "%s M=%d: no 512-row kernel (%d k-groups)", what, M, p.gk);
    CHECK(N % 512 == 0 && ksteps % 4 == 0, "%s M=%d: N %d, %d k-steps", what, M, N, ksteps);
    CHECK((long long)p.n_tg * 128 >= M && (long long)(N / 512) * p.n_tg < (1LL << 30), "%s M=%d: token groups", what, M);
  } else {
    // 33 bf16 rows and more come here only where no wide shape divides the matrix
    CHECK(!bf16 || M < kWideMinRows || N % 128, "%s M=%d: N %d left to the few-row kernel", what, M, N);
    ++n_few;
    const bool nt_ok = p.nt == 1 || p.nt == 2 || p.nt == 4 || p.nt == 8 || ((p.nt == 3 || p.nt == 6) && p.gk > 1);
    CHECK(nt_ok && (!swiglu || (p.nt % 2 == 0)), "%s M=%d: %d row tiles", what, M, p.nt);
    CHECK((p.mtt == 1 || p.mtt == 2 || (p.mtt == 4 && p.nt <= 4)), "%s M=%d: %d token tiles with %d row tiles", what,
          M, p.mtt, p.nt);
    CHECK(N % (16 * p.nt) == 0, "%s M=%d: N %d, %d row tiles", what, M, N, p.nt);
    CHECK(ksteps % (4 * p.gk) == 0, "%s M=%d: k-steps %d, %d k-groups", what, M, ksteps, p.gk);
    CHECK(p.n_tg * p.mtt * 16 >= M, "%s M=%d: token groups", what, M);
    CHECK((long long)p.n_tg * p.gk * (N / (16 * p.nt)) < (1LL << 31), "%s M=%d: grid", what, M);
  }
}

void check_matmul(const char* what, bool bf16, bool swiglu, bool allow_split, int M, int N, int K, int part_rows) {
  check_launch(what, bf16, swiglu, allow_split, M, N, K, part_rows,
               plan_mat(bf16, swiglu, M, N, K, allow_split, part_rows));
}

// Every matmul of a pass over M rows (the verify block or a prefill chunk),
// and the LM head over n_out rows.
void check_matmuls(const char* name, bool bf16, int d, int hq, int hkv, int hd, int F, int V, int M, int n_out,
                   int part_rows) {
  const int n0 = failures;
  const int nqkv = (hq + 2 * hkv) * hd;
  check_launch("qkv", bf16, false, true, M, nqkv, d, part_rows, plan_qkv(bf16, M, nqkv, d, part_rows));
  check_matmul("o", bf16, false, true, M, d, hq * hd, part_rows);
  check_matmul("gate/up", bf16, true, false, M, 2 * F, d, part_rows);
  check_matmul("down", bf16, false, true, M, d, F, part_rows);
  check_matmul("down (last, unsplit)", bf16, false, false, M, d, F, part_rows);
  if (n_out > 0) check_matmul("lm head", bf16, false, false, n_out, V, d, part_rows);
  if (failures == n0 && M % 100 == 0) std::printf("%s matmuls M=%d: ok\n", name, M);
}

// The matmuls of a model's verify passes and prefill chunks at every row
// count up to the workspace's (LM-head rows as many, up to 1024).
void check_model_matmuls(const char* name, bool bf16, int d, int hq, int hkv, int hd, int F, int V, int batch,
                         int max_block) {
  const int part_rows = cache_part_rows(batch, max_block), cap = cache_rows_cap(batch, max_block);
  for (int M = 1; M <= cap; M += M < 700 || M >= cap - 2 ? 1 : std::min(13, cap - 2 - M))
    check_matmuls(name, bf16, d, hq, hkv, hd, F, V, M, M <= 1024 ? M : 0, part_rows);
}

}  // namespace

int main() {
  const Shape s8{"8b", 32, 8, 128, true}, s14{"14b", 40, 8, 128, true}, s70{"70b", 64, 8, 128, true};
  const Shape s1{"1b", 32, 8, 64, true}, tiny{"tiny", 4, 4, 64, false};
  // the benchmark workloads (prefix lengths as drawn: the ragged batch
  // spans 512..4096)
  check_prefill(tiny, {128}, 64, 160);
  check_verify(tiny, {128}, 21, 64);
  check_prefill(s8, {1024}, 64, 1100);
  check_verify(s8, {1024}, 31, 64);
  std::vector<int> ragged;
  for (int b = 0; b < 16; ++b) ragged.push_back(512 + (b * 229) % 3585);
  ragged[3] = 4096;
  ragged[7] = 512;
  check_prefill(s8, ragged, 64, 4140);
  check_verify(s8, ragged, 31, 64);
  check_prefill(s14, std::vector<int>(4, 2048), 64, 2100);
  check_verify(s14, std::vector<int>(4, 2048), 43, 64);
  check_prefill(s70, std::vector<int>(8, 8192), 64, 8245);
  check_verify(s70, std::vector<int>(8, 8192), 45, 64);
  // edge cases: nothing to prefill, the largest batch of short prefixes
  // (segment limit), one position, a block filling max_len
  check_prefill(s70, std::vector<int>(8, 1), 64, 64);
  check_prefill(s8, std::vector<int>(256, 3), 8, 64);
  check_prefill(s8, std::vector<int>(256, 300), 8, 400);
  check_verify(s8, std::vector<int>(256, 300), 8, 8);
  check_prefill(s70, {2, 8192, 1, 4097}, 128, 8400);
  check_verify(s70, {2, 8192, 1, 4097}, 128, 128);
  // decode steps (few queries per kv head): one row per sequence, and two
  for (int S = 1; S <= 5; ++S) {
    check_verify(s1, {1024}, S, 64);
    check_verify(s1, {300, 1900, 64, 63, 65, 1, 777}, S, 64);
    check_verify(s1, std::vector<int>(16, 1100), S, 8);
    check_verify(s8, std::vector<int>(256, 4000), S, 8);
    check_verify(s70, {30000}, S, 64);
    check_verify(tiny, std::vector<int>(256, 100), S, 8);
  }
  // one long prefix among short ones: the partials are indexed by (segment,
  // query of the longest segment), more than the rows the buffer is sized for
  std::vector<int> skewed(16, 30);
  skewed[0] = 1501;
  check_prefill(s8, skewed, 31, 1600);
  skewed.assign(12, 20);
  skewed[5] = 1700;
  check_prefill(s8, skewed, 31, 1800);
  check_prefill(tiny, skewed, 31, 1800);
  skewed.assign(128, 2);
  skewed[127] = 1900;
  check_prefill(s70, skewed, 8, 2000);
  skewed.assign(100, 9);
  skewed[0] = 9000;
  check_prefill(s14, skewed, 64, 9100);
  // matmul launch shapes: the benchmark models and the tiny parity shapes, and
  // widths that the wide kernel's row groups divide partly or not at all
  check_model_matmuls("8b", true, 4096, 32, 8, 128, 14336, 128256, 256, 64);
  check_model_matmuls("8b", true, 4096, 32, 8, 128, 14336, 128256, 1, 64);
  check_model_matmuls("14b", true, 5120, 40, 8, 128, 13824, 152064, 4, 64);
  check_model_matmuls("70b", true, 8192, 64, 8, 128, 28672, 128256, 8, 64);
  check_model_matmuls("1b", true, 2048, 32, 8, 64, 8192, 128256, 16, 8);
  check_model_matmuls("tiny-f32", false, 256, 4, 4, 64, 1024, 4096, 4, 64);
  check_model_matmuls("tiny-gqa-bf16", true, 256, 8, 2, 32, 768, 4096, 8, 64);
  check_model_matmuls("d384", true, 384, 12, 12, 32, 640, 1536, 16, 72);
  check_model_matmuls("d1280-v4112", true, 1280, 10, 1, 128, 1408, 4112, 16, 72);
  check_model_matmuls("one-kv-head-of-32", true, 128, 4, 1, 32, 128, 16, 4, 64);
  if (n_wide < 1000 || n_tiled < 100 || n_few < 100) {
    std::fprintf(stderr, "plans by kernel: %lld wide, %lld 512-row, %lld few-row\n", n_wide, n_tiled, n_few);
    ++failures;
  }
  if (failures) {
    std::fprintf(stderr, "%d failure(s)\n", failures);
    return 1;
  }
  std::printf("all plans in bounds\n");
  return 0;
}
