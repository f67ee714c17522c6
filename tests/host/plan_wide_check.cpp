// CPU check of plan_wide (rv_plan.h): over the models' matrices, odd widths
// and every row count, a planned launch divides the matrix into whole row
// groups and steps, covers every row, fits the partial buffer and the grid
// limit, splits only where allowed, and leaves few rows to the few-row kernel.
#include <cstdio>
#include <vector>

#include "rv_plan.h"

int main() {
  struct Mat { int N, K; };
  const std::vector<Mat> mats = {{6144, 4096}, {4096, 4096}, {28672, 4096}, {4096, 14336}, {3072, 2048}, {2048, 2048},
                                 {16384, 2048}, {2048, 8192}, {7168, 5120}, {5120, 5120}, {27648, 5120}, {5120, 13824},
                                 {10240, 8192}, {8192, 8192}, {57344, 8192}, {8192, 28672}, {128256, 4096},
                                 {152064, 5120}, {384, 256}, {256, 768}, {1536, 256}, {1152, 384}, {1280, 1408},
                                 {128, 128}, {4096 + 16, 256}, {192, 1408}};
  long long planned = 0, bad = 0;
  for (const Mat& m : mats)
    for (int M = 1; M <= 2048; M += M < 700 ? 1 : 13)
      for (int split = 0; split < 2; ++split)
        for (int part_rows : {1024, 4096})
          for (double us : {0.0, 4.0}) {
            const WidePlan p = plan_wide(M, m.N, m.K, split != 0, part_rows, us);
            if (!p.use) continue;
            ++planned;
            const int rows = p.rows256 ? 256 : 128, ks = m.K / 32;
            const bool ok = M >= kWideMinRows && m.N % rows == 0 && p.mt >= 2 && p.mt <= 9 && p.gk >= 1 &&
                            ks % (p.gk * 2) == 0 && ks / (p.gk * 2) >= 1 && (p.gk == 1 || split) &&
                            (p.gk == 1 || (long long)p.gk * M <= part_rows) && (long long)p.n_tg * p.mt * 16 >= M &&
                            (long long)(p.n_tg - 1) * p.mt * 16 < M &&
                            (long long)(m.N / rows) * p.gk * p.n_tg < (1LL << 30);
            if (!ok && ++bad < 10)
              std::fprintf(stderr, "FAIL M=%d N=%d K=%d: rows %d mt %d n_tg %d gk %d\n", M, m.N, m.K, rows, p.mt, p.n_tg,
                           p.gk);
          }
  std::printf("%lld wide plans, %lld bad\n", planned, bad);
  return bad || planned < 1000;
}
