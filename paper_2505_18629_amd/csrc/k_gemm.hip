// Weight-streaming matrix kernel: Y[t][p] = sum_k X[t][k] W[p][k] for the
// few-token activations of a verify block (M = batch * block rows): bf16 up to
// 32 rows; with any number of them (more token groups) fp32, and bf16 widths that
// 128 does not divide (a vocabulary of any multiple of 16); and the 512-row
// kernel for hundreds of bf16 rows.
//
// Layout and schedule
//  - W is packed in 1 KiB tiles of 16 rows x KT k; activations are stored in
//    the matching operand tiles (rv_common.h).  One 16-byte load per lane
//    reads a whole tile, already in MFMA operand order.
//  - A work item is (token group of MTT tiles, row group of NT tiles, k-group
//    of K/GK).  Its 4 waves take interleaved k-steps (wave w: steps
//    kb + w, kb + w + 4, ...) so a workgroup reads one contiguous 4 KiB span
//    of every row tile per step.
//  - Each wave keeps the weight and operand tiles of its next DEPTH k-steps
//    in flight in a register ring.  Loads retire in issue order, so both
//    kinds share the ring depth.
//  - The operand tiles of a k-step are re-read (from L2) by every row group,
//    and those reads compete with the weight stream: with 2 token tiles,
//    8 row tiles per workgroup (ring depth 2) halve them relative to 4.
//  - The 4 per-wave partial tiles are summed in LDS in a fixed order.  With
//    GK > 1 the workgroup writes its fp32 partial tile and the consumer (the
//    next RMSNorm) adds the GK partials in k-group order: deterministic, no
//    atomics.
//  - bf16 models multiply every weight tile by both operand planes (hi, lo).
#include <hip/hip_ext.h>

#include "k_epilogue.h"

namespace {

constexpr int kWaves = 4;

RV_DEV uint4 load_stream(const uint4* p) {
  const u32x4 v = __builtin_nontemporal_load((const u32x4*)p);
  return uint4{v[0], v[1], v[2], v[3]};
}

template <int DT, int NT, int MTT, int EPI, int kDepth>
__global__ __launch_bounds__(kWaves * 64) void k_gemm(GemmArgs a) {
  using TR = Tr<DT>;
  constexpr int KT = TR::KT;
  constexpr int PL = DT == RV_BF16 ? 2 : 1;
  // weights are read exactly once when a single token group covers M
  constexpr bool kStream = MTT <= 2;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ksteps = a.K / KT;
  const int item = blockIdx.x;
  const int tg = item % a.n_tg, rest = item / a.n_tg;
  const int kg = rest % a.gk, rg = rest / a.gk;
  const int kb = kg * (ksteps / a.gk);
  const int spr = ksteps / (a.gk * kWaves);  // k-steps per wave
  const int tile0 = rg * NT;
  const int tok0 = tg * MTT * 16;

  const uint4* wp = (const uint4*)a.W + (size_t)tile0 * ksteps * 64 + (size_t)(kb + w) * 64 + lane;
  const uint4* xp[PL];
#pragma unroll
  for (int pl = 0; pl < PL; ++pl)
    xp[pl] = (const uint4*)(pl ? a.X2 : a.X) + (size_t)(tok0 >> 4) * ksteps * 64 + (size_t)(kb + w) * 64 + lane;

  f32x4_t acc[NT][MTT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int mt = 0; mt < MTT; ++mt) acc[nt][mt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  uint4 wq[kDepth][NT], xq[kDepth][PL][MTT];
  // the j-th k-step of this wave is kb + w + 4j
  auto load = [&](int slot, int j) {
    const size_t o = (size_t)j * (kWaves * 64);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const uint4* p = wp + (size_t)nt * ksteps * 64 + o;
      wq[slot][nt] = kStream ? load_stream(p) : *p;
    }
#pragma unroll
    for (int pl = 0; pl < PL; ++pl)
#pragma unroll
      for (int mt = 0; mt < MTT; ++mt) xq[slot][pl][mt] = xp[pl][(size_t)mt * ksteps * 64 + o];
  };
  auto compute = [&](int slot) {
#pragma unroll
    for (int pl = 0; pl < PL; ++pl)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < MTT; ++mt) mma_step<DT>(wq[slot][nt], xq[slot][pl][mt], acc[nt][mt]);
  };
  // Full groups of kDepth steps run branch-free; the last full group only
  // computes; a remainder (spr not a multiple of kDepth) runs unpipelined.
  const int nfull = spr / kDepth;
  int j = 0;
  if (nfull > 0) {
#pragma unroll
    for (int d = 0; d < kDepth; ++d) load(d, d);
    for (int gi = 1; gi < nfull; ++gi) {
#pragma unroll
      for (int d = 0; d < kDepth; ++d) {
        compute(d);
        load(d, j + kDepth + d);
      }
      j += kDepth;
    }
#pragma unroll
    for (int d = 0; d < kDepth; ++d) compute(d);
    j += kDepth;
  }
  for (; j < spr; ++j) {
    load(0, j);
    compute(0);
  }

  __shared__ f32x4_t red[kWaves][NT][MTT][64];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int mt = 0; mt < MTT; ++mt) red[w][nt][mt][lane] = acc[nt][mt];
  __syncthreads();
  for (int mt = w; mt < MTT; mt += kWaves) {
    f32x4_t v[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      v[nt] = red[0][nt][mt][lane];
#pragma unroll
      for (int ww = 1; ww < kWaves; ++ww) v[nt] += red[ww][nt][mt][lane];
    }
    const int tok = tok0 + mt * 16 + (lane & 15);
    EpiLoad<EPI, NT> ld;
    epilogue_load<NT, EPI>(a, tile0, tok, lane, ld);
    epilogue<DT, NT, EPI>(a, tile0, kg, tok, lane, v, ld);
  }
}

// ------------------------------------------------------------ many tokens
// bf16, hundreds of rows and more (long prefill chunks, large batches of
// matrices whose rows fill whole 512-row groups): a workgroup owns 512 output
// rows x 128 tokens.  Its 8 waves (two per SIMD, so one wave's LDS and load
// waits overlap the other's MFMAs) take 4 row tiles each and share the 8
// token tiles: each k-step's operand tiles (hi and lo) are staged once per
// workgroup in double-buffered LDS.  Weight tiles go straight to registers.
// Both are fetched DEPTH k-steps ahead through a register ring.  The operand
// tiles of a k-step are read from LDS in chunks of CH, chunk i+1 before the
// MFMAs of chunk i; without the scheduling barriers the compiler reads two
// tiles, waits for both and only then multiplies, so every pair exposes the
// LDS latency (8B gate/up at 496 tokens 189 - 211 -> 183 - 188 us; CH = 4
// spills).  Workgroups that share rows (the token groups of a row group) have
// consecutive items on one XCD, so the weights come from HBM about once.
// Every load index is clamped, so the pipeline has no branches; rows past M
// are computed and not stored.  Bound by MFMA power: 1.26 - 1.51 PFLOP/s of
// hi/lo products at 496 - 2047 tokens (8B gate/up 180, 346 and 696 us at 496, 1024
// and 2047; 70B 701, 1389 and 2540), where a large library bf16 product of
// random data reaches 1.25 - 1.48 on this part.
template <int EPI>
__global__ __launch_bounds__(512) void k_gemm_tiled(GemmArgs a, int items) {
  constexpr int NT = 4, MT = 8, NW = 8, DEPTH = 4, CH = 2, NCH = 2 * MT / CH;
  constexpr int XU = MT * 2 * 64 / (NW * 64);  // 16-byte operand chunks per thread and k-step
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ks = a.K / 32;
  const int item = xcd_item(blockIdx.x, items);
  if (item >= items) return;
  const int tg = item % a.n_tg, rg = item / a.n_tg;
  const int tile0 = (rg * NW + w) * NT;  // this wave's first row tile
  const int last_tt = (a.M - 1) >> 4;    // last valid token tile

  const u32x4* wp = (const u32x4*)a.W + (size_t)tile0 * ks * 64 + lane;
  // operand chunk u of this thread: plane, token tile, lane slot
  const u32x4* xsrc[XU];
#pragma unroll
  for (int u = 0; u < XU; ++u) {
    const int c = threadIdx.x + u * NW * 64;
    const int pl = c / (MT * 64), m = (c / 64) % MT, l16 = c % 64;
    const int tt = min(tg * MT + m, last_tt);
    xsrc[u] = (const u32x4*)(pl ? a.X2 : a.X) + (size_t)tt * ks * 64 + l16;
  }
  __shared__ u32x4 xs[2][2 * MT * 64];

  f32x4_t acc[NT][MT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  u32x4 wq[DEPTH][NT], xq[DEPTH][XU];
  auto load = [&](int slot, int step) {
    step = min(step, ks - 1);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) wq[slot][nt] = wp[((size_t)nt * ks + step) * 64];
#pragma unroll
    for (int u = 0; u < XU; ++u) xq[slot][u] = xsrc[u][(size_t)step * 64];
  };
  auto stage = [&](int slot, int buf) {
#pragma unroll
    for (int u = 0; u < XU; ++u) xs[buf][threadIdx.x + u * NW * 64] = xq[slot][u];
  };
  auto compute = [&](int slot, int buf) {
    bf16x8_t xr[2][CH];
    auto read = [&](int i) {
#pragma unroll
      for (int c = 0; c < CH; ++c) xr[i & 1][c] = __builtin_bit_cast(bf16x8_t, xs[buf][(i * CH + c) * 64 + lane]);
    };
    read(0);
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      if (i + 1 < NCH) read(i + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          acc[nt][(i * CH + c) % MT] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8_t, wq[slot][nt]), xr[i & 1][c], acc[nt][(i * CH + c) % MT], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

#pragma unroll
  for (int d = 0; d < DEPTH; ++d) load(d, d);
  stage(0, 0);
  __syncthreads();
  // Step d of a ring turn: the next step's operands go to the other LDS
  // buffer, this step is computed, and its ring slot fetches the step DEPTH
  // ahead.
  for (int s0 = 0; s0 < ks; s0 += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      stage((d + 1) % DEPTH, (d & 1) ^ 1);
      compute(d, d & 1);
      load(d, s0 + d + DEPTH);
      __syncthreads();
    }
  }

  epilogue_tiles<RV_BF16, NT, EPI, MT, 2>(a, tile0, 0, tg * MT * 16 + (lane & 15), lane, acc, 0, MT);
}

template <int DT, int NT, int MTT, int EPI>
void launch_one(const GemmArgs& a, unsigned items, hipStream_t st) {
  constexpr int kDepth = NT >= 6 ? 2 : 4;
  const dim3 block(kWaves * 64);
  LaunchEvents& ev = g_launch_events;
  if (ev.start) {
    hipExtLaunchKernelGGL(k_gemm<DT, NT, MTT, EPI, kDepth>, dim3(items), block, 0, st, ev.start, ev.stop, 0, a);
    ev = LaunchEvents{};
  } else {
    k_gemm<DT, NT, MTT, EPI, kDepth><<<items, block, 0, st>>>(a);
  }
}

template <int DT, int NT, int EPI>
hipError_t launch_nt(const GemmArgs& a, int mtt, hipStream_t st) {
  const unsigned items = (unsigned)(a.n_tg * a.gk * (a.N / (16 * NT)));
  switch (mtt) {
    case 1: launch_one<DT, NT, 1, EPI>(a, items, st); break;
    case 2: launch_one<DT, NT, 2, EPI>(a, items, st); break;
    case 4:
      if constexpr (NT <= 4) {
        launch_one<DT, NT, 4, EPI>(a, items, st);
        break;
      }
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int DT, int EPI>
hipError_t launch_epi(const GemmArgs& a, int nt, int mtt, hipStream_t st) {
  switch (nt) {
    case 1:
      if constexpr (EPI != EPI_SWIGLU) return launch_nt<DT, 1, EPI>(a, mtt, st);
      break;
    case 2: return launch_nt<DT, 2, EPI>(a, mtt, st);
    case 4: return launch_nt<DT, 4, EPI>(a, mtt, st);
    case 8: return launch_nt<DT, 8, EPI>(a, mtt, st);
    case 3:
    case 6:
      // only K-split launches use 3 or 6 row tiles
      if constexpr (EPI == EPI_PARTIAL) return nt == 3 ? launch_nt<DT, 3, EPI>(a, mtt, st)
                                                       : launch_nt<DT, 6, EPI>(a, mtt, st);
      break;
  }
  return hipErrorInvalidValue;
}

template <int DT>
hipError_t launch_dt(int epi, const GemmArgs& a, int nt, int mtt, hipStream_t st) {
  switch (epi) {
    case EPI_STORE: return launch_epi<DT, EPI_STORE>(a, nt, mtt, st);
    case EPI_RESID: return launch_epi<DT, EPI_RESID>(a, nt, mtt, st);
    case EPI_PARTIAL: return launch_epi<DT, EPI_PARTIAL>(a, nt, mtt, st);
    case EPI_SWIGLU: return launch_epi<DT, EPI_SWIGLU>(a, nt, mtt, st);
    case EPI_QKV: return launch_epi<DT, EPI_QKV>(a, nt, mtt, st);
    case EPI_STORE_LOGICAL: return launch_epi<DT, EPI_STORE_LOGICAL>(a, nt, mtt, st);
  }
  return hipErrorInvalidValue;
}

template <int EPI>
hipError_t launch_tiled_epi(const GemmArgs& a, hipStream_t st) {
  const int items = a.N / 512 * a.n_tg;
  const unsigned grid = (unsigned)((items + 7) / 8 * 8);
  LaunchEvents& ev = g_launch_events;
  if (ev.start) {
    hipExtLaunchKernelGGL(k_gemm_tiled<EPI>, dim3(grid), dim3(512), 0, st, ev.start, ev.stop, 0, a, items);
    ev = LaunchEvents{};
  } else {
    k_gemm_tiled<EPI><<<grid, 512, 0, st>>>(a, items);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_tiled(int epi, const GemmArgs& a, hipStream_t st) {
  if (a.gk != 1 || (a.K / 32) % 4 || a.N % 512 || (long long)a.n_tg * 128 < a.M) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_STORE: return launch_tiled_epi<EPI_STORE>(a, st);
    case EPI_RESID: return launch_tiled_epi<EPI_RESID>(a, st);
    case EPI_SWIGLU: return launch_tiled_epi<EPI_SWIGLU>(a, st);
    case EPI_QKV: return launch_tiled_epi<EPI_QKV>(a, st);
    case EPI_STORE_LOGICAL: return launch_tiled_epi<EPI_STORE_LOGICAL>(a, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_wide(int epi, const GemmArgs& a, bool rows256, int mt, hipStream_t st) {
  if (a.gk < 1 || (a.K / 32) % (2 * a.gk) || a.N % (rows256 ? 256 : 128) || (long long)a.n_tg * mt * 16 < a.M)
    return hipErrorInvalidValue;
  if (a.gk > 1 && epi != EPI_PARTIAL) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_STORE: return launch_wide_store(a, rows256, mt, st);
    case EPI_RESID: return launch_wide_resid(a, rows256, mt, st);
    case EPI_PARTIAL: return launch_wide_partial(a, rows256, mt, st);
    case EPI_SWIGLU: return launch_wide_swiglu(a, rows256, mt, st);
    case EPI_QKV: return launch_wide_qkv(a, rows256, mt, st);
    case EPI_STORE_LOGICAL: return launch_wide_store_logical(a, rows256, mt, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm(int dtype, int epi, const GemmArgs& a, int nt, int mtt, hipStream_t st) {
  return dtype == RV_BF16 ? launch_dt<RV_BF16>(epi, a, nt, mtt, st) : launch_dt<RV_F32>(epi, a, nt, mtt, st);
}
