// Matrix kernel for 33 rows and more (bf16): Y[t][p] = sum_k X[t][k] W[p][k].
//
// A workgroup owns RW x NT row tiles x MT token tiles of one k-group: all the
// tokens, or one of several groups of them, as plan_wide estimates cheaper.  Its
// waves have two roles:
//  - RW x KW consumer waves: wave (rw, kw) multiplies NT row tiles by the MT
//    token tiles at the k-steps kw, kw + KW, ...; its weights go straight from
//    global memory to a register ring DEPTH k-steps deep.
//  - PW producer waves copy the operand tiles (hi and lo planes) of the next
//    steps into a ring of NB LDS buffers with 16-byte direct loads.  Their
//    barriers leave copies in flight (with __syncthreads every copy had to land
//    before the next barrier: 14B gate/up at 172 rows 109 -> 98 us, 8B down at
//    203 rows 53 -> 52, 70B gate/up at 360 rows 597 -> 548, with two k-steps per
//    barrier).
// Loads of one wave retire in issue order, so a wave that fetched both
// operands and weights would hold the weight stream to the operand ring's
// depth; with the roles apart each keeps its own.
//
// Step s covers the k-steps 2s and 2s+1 of the k-group (with KW = 1 every
// consumer takes both: against one k-step per barrier 1 - 5% at 172 - 2047
// rows, 8B O at 2047 102.8 -> 97.2 us).  Barrier s: the
// operands of steps s and s+1 are in LDS, and the buffer of step s-1 is free.
// Having step s+1 early lets a consumer read the first operand chunk of the
// next step before the barrier that ends this one; chunk i+1 is always read
// before the MFMAs of chunk i (scheduling barriers keep that order -- left
// alone, the compiler waits for every pair of LDS reads right before its
// MFMAs).
//
// What bounds it: every workgroup re-reads the operand rows (4 bytes per
// element and row) from L2 beside its own weights, so up to about 100 rows the
// limit is the sum of both streams, beyond that MFMA power.  Measured against
// the kernel before it (8 waves, operand tiles of 64 - 128 tokens through
// registers; us per launch, partial sums' traffic not counted):
//   8B   93 rows: gate/up 68 -> 53, down 55 -> 30, O 20 -> 13, QKV 21.7 -> 19.6
//   14B 172 rows: gate/up 112 -> 104, down 62 -> 58 (with 6 k-groups)
//   8B  203 rows: gate/up 109 -> 89, down 57 -> 49
//   70B 360 rows: gate/up 603 -> 549;  LM head, 144 rows of 8192: 711 -> 498
//   LM head, 36 rows of 4096: 255 -> 189;  1B 716 rows: O 45 -> 16
// Nontemporal weight loads where one token group covers every row (each
// weight is then read once): 57 -> 54 us at 8B gate/up, 212 -> 189 at the LM
// head; with several groups the other groups' reads hit L2, so plain loads.
#pragma once
#include <hip/hip_ext.h>

#include "k_epilogue.h"

namespace {

constexpr int kWideProducers = 4;
constexpr int kWideLdsUnits = 160;  // 1 KiB operand tiles that fit the 160 KiB of LDS

constexpr int cmin(int a, int b) { return a < b ? a : b; }
constexpr int cmax(int a, int b) { return a > b ? a : b; }

template <int NT, int MT, int RW, int KW>
struct WideCfg {
  static constexpr int PW = kWideProducers;
  static constexpr int THREADS = (RW * KW + PW) * 64;
  static constexpr int DEPTH = 4;                        // weight ring, k-steps of a wave
  static constexpr int CH = NT * MT >= 32 || MT == 9 ? 2 : 4;      // operand tiles per LDS read chunk (registers)
  static constexpr int NCH = (2 * MT + CH - 1) / CH;
  static constexpr int KPB = 2 / KW;                     // k-steps of a wave per step
  static constexpr int UNITS = 2 * MT * 2;               // operand tiles of a step (two k-steps, two planes)
  static constexpr int U = (UNITS + PW - 1) / PW;        // copies per producer wave and step
  static constexpr int NB = cmin(6, kWideLdsUnits / UNITS);  // LDS buffers
  static constexpr int RED = KW > 1 ? RW * NT * MT : 0;  // tiles exchanged by the k-halves
  static_assert(NB >= 3, "steps s and s+1 resident, s+2 in flight");
  static_assert((NB - 1) * U <= 63, "copies in flight must fit the load counter");
  static_assert(KW == 1 || KW == 2, "the k-halves exchange accumulators pairwise");
  static constexpr int LDS = cmax(NB * UNITS, RED) * 64;
};

template <int NT, int MT, int RW, int KW, bool STREAM, int EPI>
__global__ __launch_bounds__((WideCfg<NT, MT, RW, KW>::THREADS)) void k_gemm_wide(GemmArgs a, int items) {
  using C = WideCfg<NT, MT, RW, KW>;
  constexpr int DEPTH = C::DEPTH, CH = C::CH, NCH = C::NCH, KPB = C::KPB, UNITS = C::UNITS, NB = C::NB;
  __shared__ u32x4 xs[C::LDS];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ksteps = a.K / 32;
  // Item = (row group, k-group) x token group; the token groups of one
  // (row group, k-group) are consecutive items, on one XCD.
  const int item = xcd_item(blockIdx.x, items);
  if (item >= items) return;
  const int tg = item % a.n_tg, rk = item / a.n_tg;
  const int rg = rk / a.gk, kg = rk % a.gk;
  const int kb = kg * (ksteps / a.gk), ss = ksteps / (a.gk * 2);  // first k-step, steps

  if (w >= RW * KW) {
    // ---- producer
    const int p = w - RW * KW, last_tt = (a.M - 1) >> 4;
    const u32x4* src[C::U];
    int dst[C::U];
#pragma unroll
    for (int u = 0; u < C::U; ++u) {
      const int un = min(p + u * C::PW, UNITS - 1);  // past the last unit: it again
      const int kk = un / (MT * 2), pl = un / MT % 2, m = un % MT;
      const int tt = min(tg * MT + m, last_tt);
      src[u] = (const u32x4*)(pl ? a.X2 : a.X) + ((size_t)tt * ksteps + kb + kk) * 64 + lane;
      dst[u] = un * 64;
    }
    auto fetch = [&](int s, int buf) {
      s = min(s, ss - 1);  // past the end: a valid step, not read
#pragma unroll
      for (int u = 0; u < C::U; ++u)
        __builtin_amdgcn_global_load_lds((const void*)(src[u] + (size_t)s * 128),
                                         (__attribute__((address_space(3))) void*)(&xs[buf * UNITS * 64 + dst[u]]), 16,
                                         0, 0);
    };
    for (int i = 0; i < NB - 1; ++i) fetch(i, i);
    int buf = NB - 1;
    for (int s = 0; s < ss; ++s) {
      __builtin_amdgcn_s_waitcnt(wait_vm((NB - 3) * C::U));  // this wave's copies of steps <= s + 1 have landed
      barrier_keep_loads();                                  // barrier s
      fetch(s + NB - 1, buf);                                // into the buffer of step s - 1
      buf = buf == NB - 1 ? 0 : buf + 1;
    }
    __builtin_amdgcn_s_waitcnt(wait_vm(0));
    __syncthreads();  // barrier ss
    if constexpr (KW > 1) __syncthreads();
    return;
  }

  // ---- consumer
  const int kw = w % KW, rw = w / KW;
  const int tile0 = (rg * RW + rw) * NT;
  const u32x4* wp = (const u32x4*)a.W + ((size_t)tile0 * ksteps + kb + kw) * 64 + lane;
  f32x4_t acc[NT][MT];
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[n][m] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  u32x4 wq[DEPTH][NT];
  // the j-th k-step of this wave is kb + kw + j KW
  auto load = [&](int slot, int j) {
    j = min(j, ss * KPB - 1);
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const u32x4* p = wp + ((size_t)n * ksteps + (size_t)j * KW) * 64;
      wq[slot][n] = STREAM ? __builtin_nontemporal_load(p) : *p;
    }
  };
  // operand tile t of k-step sub of a step: plane t / MT, token tile t % MT
  bf16x8_t xr[2][CH];
  const u32x4* xbase = &xs[kw * MT * 2 * 64 + lane];
  auto read = [&](int par, int sub, int i, int buf) {
#pragma unroll
    for (int c = 0; c < CH; ++c)
      if (i * CH + c < 2 * MT)
        xr[par][c] = __builtin_bit_cast(bf16x8_t, xbase[(buf * UNITS + sub * 2 * MT + i * CH + c) * 64]);
  };
  auto multiply = [&](int par, int i, int slot) {
#pragma unroll
    for (int c = 0; c < CH; ++c)
      if (i * CH + c < 2 * MT) {
        const int m = (i * CH + c) % MT;
#pragma unroll
        for (int n = 0; n < NT; ++n)
          acc[n][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wq[slot][n]), xr[par][c],
                                                             acc[n][m], 0, 0, 0);
      }
  };
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) load(d, d);
  int buf = 0, s = 0;
  // One step, the d-th of a turn of the ring; chunk 0 of its operands was read
  // before.
  auto step = [&](int d, bool more) {
    const int next = buf == NB - 1 ? 0 : buf + 1;
#pragma unroll
    for (int sub = 0; sub < KPB; ++sub) {
      const int slot = d * KPB + sub;
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        const int par = (slot * NCH + i) & 1;
        if (i + 1 < NCH) read(par ^ 1, sub, i + 1, buf);
        else if (sub + 1 < KPB) read(par ^ 1, sub + 1, 0, buf);
        else read(par ^ 1, 0, 0, next);  // after the last step: read and not used
        __builtin_amdgcn_sched_barrier(0);
        multiply(par, i, slot);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (more) load(slot, (s + d) * KPB + sub + DEPTH);
      __builtin_amdgcn_sched_barrier(0);
    }
    buf = next;
    __syncthreads();  // barrier s + d + 1
  };
  __syncthreads();  // barrier 0
  read(0, 0, 0, 0);
  constexpr int TURN = DEPTH / KPB;
  for (; s + TURN <= ss; s += TURN) {
#pragma unroll
    for (int d = 0; d < TURN; ++d) step(d, true);
  }
#pragma unroll
  for (int d = 0; d < TURN - 1; ++d)
    if (s + d < ss) step(d, false);

  // The two k-halves of a row tile add up: each gives the other half of its
  // token tiles (through the LDS ring, which is idle now) and finishes its own.
  const int tok0 = tg * MT * 16 + (lane & 15);
  if constexpr (KW > 1) {
    constexpr int H = (MT + 1) / 2;
    f32x4_t* red = (f32x4_t*)xs + (size_t)rw * NT * MT * 64 + lane;
    const bool first = kw == 0;
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int m = 0; m < MT; ++m)
        if (first == (m >= H)) red[(n * MT + m) * 64] = acc[n][m];
    __syncthreads();
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int m = 0; m < MT; ++m)
        if (first == (m < H)) acc[n][m] += red[(n * MT + m) * 64];
    if (first) epilogue_tiles<RV_BF16, NT, EPI, MT, H>(a, tile0, kg, tok0, lane, acc, 0, H);
    else epilogue_tiles<RV_BF16, NT, EPI, MT, H>(a, tile0, kg, tok0, lane, acc, H, MT);
  } else {
    epilogue_tiles<RV_BF16, NT, EPI, MT, EPI == EPI_QKV ? 2 : 3>(a, tile0, kg, tok0, lane, acc, 0, MT);
  }
}

template <int NT, int MT, int RW, int KW, int EPI>
hipError_t launch_wide_one(const GemmArgs& a, hipStream_t st) {
  const int items = a.N / (16 * NT * RW) * a.gk * a.n_tg;
  const dim3 grid((unsigned)((items + 7) / 8 * 8)), block(WideCfg<NT, MT, RW, KW>::THREADS);
  const auto kernel = a.n_tg == 1 ? k_gemm_wide<NT, MT, RW, KW, true, EPI> : k_gemm_wide<NT, MT, RW, KW, false, EPI>;
  LaunchEvents& ev = g_launch_events;
  if (ev.start) {
    hipExtLaunchKernelGGL(kernel, grid, block, 0, st, ev.start, ev.stop, 0, a, items);
    ev = LaunchEvents{};
  } else {
    kernel<<<grid, block, 0, st>>>(a, items);
  }
  return hipGetLastError();
}

template <int MT, int EPI>
hipError_t launch_wide_mt(const GemmArgs& a, bool rows256, hipStream_t st) {
  return rows256 ? launch_wide_one<4, MT, 4, 1, EPI>(a, st) : launch_wide_one<2, MT, 4, 2, EPI>(a, st);
}

template <int EPI>
hipError_t launch_wide_epi(const GemmArgs& a, bool rows256, int mt, hipStream_t st) {
  switch (mt) {
    case 2: return launch_wide_mt<2, EPI>(a, rows256, st);
    case 3: return launch_wide_mt<3, EPI>(a, rows256, st);
    case 4: return launch_wide_mt<4, EPI>(a, rows256, st);
    case 5: return launch_wide_mt<5, EPI>(a, rows256, st);
    case 6: return launch_wide_mt<6, EPI>(a, rows256, st);
    case 7: return launch_wide_mt<7, EPI>(a, rows256, st);
    case 8: return launch_wide_mt<8, EPI>(a, rows256, st);
    case 9: return launch_wide_mt<9, EPI>(a, rows256, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace
