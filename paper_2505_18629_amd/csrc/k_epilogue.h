// Epilogues of the matrix kernels: what a wave does with the finished 16-row
// tiles of one token (lane l holds rows 4(l/16)..+3 of token l%16).
#pragma once
#include "rv_internal.h"

namespace {

RV_DEV float silu(float g) { return g / (1.0f + __expf(-g)); }

// What an epilogue reads: the residual rows it adds to, or the rotary factors
// and the cache place of the token.  Callers with several token tiles load
// them for a batch of tiles first and then finish the batch: with load and
// store in turn every tile would expose one (residual) or two (position, then
// rotary factors) memory latencies -- 12 us of the 62 us of the 8B QKV at 496
// tokens, 27 us of the 90 us of the 1B O and down at 716.
template <int EPI, int NT>
struct EpiLoad {};
template <int NT>
struct EpiLoad<EPI_RESID, NT> {
  f32x4_t y[NT];
};
template <int NT>
struct EpiLoad<EPI_QKV, NT> {
  int pos, seq;
  f32x4_t cs[NT], sn[NT];
};

// Loads of token tok (clamped to the last token).
template <int NT, int EPI>
RV_DEV void epilogue_load(const GemmArgs& a, int tile0, int tok, int lane, EpiLoad<EPI, NT>& ld) {
  const int g = lane >> 4, t = min(tok, a.M - 1);
  if constexpr (EPI == EPI_RESID) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) ld.y[nt] = *(const f32x4_t*)(a.Y + (size_t)t * a.ldy + (tile0 + nt) * 16 + 4 * g);
  } else if constexpr (EPI == EPI_QKV) {
    ld.pos = a.row_pos[t];
    ld.seq = a.row_seq[t];
    // tile j of a head holds dims 8j..8j+7 (rows 0..7) and their partners; v
    // tiles load the factors of the same place and do not use them
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int j = ((tile0 + nt) * 16 % a.hd) >> 4;
      const size_t o = (size_t)ld.pos * (a.hd >> 1) + 8 * j + 4 * (g & 1);
      ld.cs[nt] = *(const f32x4_t*)(a.rope_cos + o);
      ld.sn[nt] = *(const f32x4_t*)(a.rope_sin + o);
    }
  }
}

template <int DT, int NT, int EPI>
RV_DEV void epilogue(const GemmArgs& a, int tile0, int kg, int tok, int lane, f32x4_t (&v)[NT],
                     const EpiLoad<EPI, NT>& ld) {
  const int g = lane >> 4;
  if constexpr (EPI == EPI_STORE || EPI == EPI_RESID) {
    if (tok >= a.M) return;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      f32x4_t r = v[nt];
      if constexpr (EPI == EPI_RESID) r += ld.y[nt];
      *(f32x4_t*)(a.Y + (size_t)tok * a.ldy + (tile0 + nt) * 16 + 4 * g) = r;
    }
  } else if constexpr (EPI == EPI_PARTIAL) {
    if (tok >= a.M) return;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
      *(f32x4_t*)(a.P + ((size_t)kg * a.M + tok) * a.ldy + (tile0 + nt) * 16 + 4 * g) = v[nt];
  } else if constexpr (EPI == EPI_STORE_LOGICAL) {
    if (tok >= a.M) return;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int p = (tile0 + nt) * 16 + 4 * g + i;
        a.Y[(size_t)tok * a.ldy + mat_logical_row(a.md, p)] = v[nt][i];
      }
  } else if constexpr (EPI == EPI_SWIGLU) {
    // physical tile 2t holds gate rows, 2t+1 the matching up rows
    if (tok >= a.M) return;
#pragma unroll
    for (int nt = 0; nt < NT; nt += 2) {
      const int f0 = ((tile0 + nt) >> 1) * 16 + 4 * g;
      f32x4_t out;
#pragma unroll
      for (int i = 0; i < 4; ++i) out[i] = silu(v[nt][i]) * v[nt + 1][i];
      put_operand4<DT>(a.act, a.act2, tok, f0, a.N / 2, out);
    }
  } else if constexpr (EPI == EPI_QKV) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      // Rotate-half partner of row r (r < 8) is row r + 8, held by lane ^ 32.
      f32x4_t partner;
#pragma unroll
      for (int i = 0; i < 4; ++i) partner[i] = __shfl_xor(v[nt][i], 32, 64);
      if (tok >= a.M) continue;
      const int p0 = (tile0 + nt) * 16;
      if (p0 < a.q_rows + a.k_rows) {
        const bool is_q = p0 < a.q_rows;
        const int rel = is_q ? p0 : p0 - a.q_rows;
        const int head = rel / a.hd, j = (rel % a.hd) >> 4;
        const bool second = lane >= 32;
        f32x4_t rot;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float c = ld.cs[nt][i], s = ld.sn[nt][i];
          rot[i] = second ? v[nt][i] * c + partner[i] * s : v[nt][i] * c - partner[i] * s;
        }
        const int dim = (second ? a.hd >> 1 : 0) + 8 * j + 4 * (g & 1);
        if (is_q) {
          put_operand4<DT>(a.qbuf, a.qbuf2, tok, head * a.hd + dim, a.n_heads * a.hd, rot);
        } else {
          put_k4<DT>(a.kc, a.kc2, (size_t)(ld.seq * a.n_kv + head) * a.kv_len * a.hd, ld.pos, dim, a.hd, rot);
        }
      } else {
        const int rel = p0 - a.q_rows - a.k_rows + 4 * g;
        const int head = rel / a.hd, dim = rel % a.hd;
        put_v4<DT>(a.vc, a.vc2, (size_t)(ld.seq * a.n_kv + head) * a.kv_len * a.hd, ld.pos, dim, a.hd, v[nt]);
      }
    }
  }
}

// Token tiles [m0, m1) of acc, in batches of EB: all of a batch's loads, then
// its stores.  m0, m1: constants after unrolling.
template <int DT, int NT, int EPI, int MT, int EB>
RV_DEV void epilogue_tiles(const GemmArgs& a, int tile0, int kg, int tok0, int lane, f32x4_t (&acc)[NT][MT], int m0,
                           int m1) {
#pragma unroll
  for (int b0 = 0; b0 < MT; b0 += EB) {
    EpiLoad<EPI, NT> ld[EB];
#pragma unroll
    for (int e = 0; e < EB; ++e)
      if (m0 + b0 + e < m1) epilogue_load<NT, EPI>(a, tile0, tok0 + (m0 + b0 + e) * 16, lane, ld[e]);
#pragma unroll
    for (int e = 0; e < EB; ++e)
      if (m0 + b0 + e < m1) {
        f32x4_t v[NT];
#pragma unroll
        for (int n = 0; n < NT; ++n) v[n] = acc[n][m0 + b0 + e];
        epilogue<DT, NT, EPI>(a, tile0, kg, tok0 + (m0 + b0 + e) * 16, lane, v, ld[e]);
      }
  }
}

}  // namespace
