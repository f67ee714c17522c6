// k_gemm_wide with the EPI_RESID epilogue (one file per epilogue: they compile in parallel).
#include "k_wide.h"

hipError_t launch_wide_resid(const GemmArgs& a, bool rows256, int mt, hipStream_t st) {
  return launch_wide_epi<EPI_RESID>(a, rows256, mt, st);
}
