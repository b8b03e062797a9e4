// The scalar body of the general path of fused-RoPE paged attention (§3.3.3): a workgroup serves up to GM query heads of one
// (query token, KV head, range of slots) with plain fp32 arithmetic. The path's matrix-core kernels fall back to it for a
// token whose result came out NaN or Inf: operands split into two bf16 terms turn some infinities (0 x Inf, Inf - Inf between the
// terms) into NaN where plain arithmetic has none, matrix products bring slots together that a row must not see, and
// probabilities relative to a reference that lags the maximum overflow earlier than the body's, which are at most 1.
//
// Per tile of kThreads slots:
//   phase A  thread = slot: gather the K row through the block table, rotate it at the slot's
//            absolute position, dot it with the rotated queries (LDS broadcast) -> scores in LDS;
//   softmax  online max / sum per head with wave shuffles + one LDS exchange;
//   phase B  thread = (dim, part): walk the tile's V rows (contiguous per dim in the V page layout)
//            and accumulate p * v for the heads.
#pragma once
#include "attn_common.h"

namespace mepic {

template <int KV> struct Store;
template <> struct Store<MEPIC_F32> { using T = float; static constexpr int X = 4; };
template <> struct Store<MEPIC_BF16> { using T = uint16_t; static constexpr int X = 8; };
template <> struct Store<MEPIC_F8E4M3> { using T = uint8_t; static constexpr int X = 16; };

// Load one 16-byte granule and widen it to fp32.
template <int KV>
__device__ __forceinline__ void load_granule(const void* base, size_t granule_index, float* x) {
  const uint4 w = reinterpret_cast<const uint4*>(base)[granule_index];
  const uint32_t u[4] = {w.x, w.y, w.z, w.w};
  if constexpr (KV == MEPIC_F32) {
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(u[i]);
  } else if constexpr (KV == MEPIC_BF16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = bf16_bits_to_f32(u[i] & 0xffffu);
      x[2 * i + 1] = bf16_bits_to_f32(u[i] >> 16);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int k = 0; k < 4; ++k) x[4 * i + k] = e4m3_to_f32((u[i] >> (8 * k)) & 0xffu);
  }
}

__device__ __forceinline__ float load_q(const void* q, int q_dtype, size_t idx) {
  return q_dtype == MEPIC_F32 ? reinterpret_cast<const float*>(q)[idx]
                              : bf16_bits_to_f32(reinterpret_cast<const uint16_t*>(q)[idx]);
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

template <int GM, int kThreads>
struct ScalarLds {
  float qhat[GM * 2 * kMaxHalfD];       // [G][D], rotated, pre-multiplied by the score scale
  float sc[GM * kThreads];              // [G][kThreads] scores, then probabilities, of the tile
  float red[kThreads / 64 * GM];
  unsigned char took[kThreads];         // does the slot of the tile take part (valid, visible, below kv_len)?
};

// GM: compile-time bound on G, the heads g0 .. g0 + G - 1 of KV head hk this call serves, so that per-head arrays stay in
// registers. Slots [n_begin, n_end) of request b for query token t; n_begin is a multiple of P. The result goes to the
// partials of `split`, or, if `direct`, normalised to the output row. Every thread of the workgroup calls.
template <int KV, int GM, int kThreads>
__device__ __forceinline__ void scalar_attend(const AttnArgs& a, ScalarLds<GM, kThreads>& lds, int t, int b, int hk, int g0,
                                              int G, int n_begin, int n_end, int split, bool direct) {
  constexpr int X = Store<KV>::X, kWaves = kThreads / 64;
  using T = typename Store<KV>::T;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int D = a.D, P = a.P, half = D / 2;
  const int pos_q = a.q_positions[t];

  // rotate the G queries of this KV head at the query's own position
  for (int idx = tid; idx < G * half; idx += kThreads) {
    const int g = idx / half, i = idx % half;
    const int i0 = a.interleaved ? 2 * i : i, i1 = a.interleaved ? 2 * i + 1 : i + half;
    const size_t base = ((size_t)t * a.Hq + (size_t)hk * a.G + g0 + g) * D;
    const float x0 = load_q(a.q, a.q_dtype, base + i0), x1 = load_q(a.q, a.q_dtype, base + i1);
    float sn, cs;
    sincospif(2.0f * turns_frac((float)pos_q, a.freq_hi[i], a.freq_lo[i]), &sn, &cs);
    lds.qhat[g * D + i0] = (x0 * cs - x1 * sn) * a.qk_scale_log2;
    lds.qhat[g * D + i1] = (x1 * cs + x0 * sn) * a.qk_scale_log2;
  }
  __syncthreads();

  // phase-B ownership: dim d, and every `parts`-th block of the tile
  const int d_own = tid % D, part = tid / D, parts = kThreads / D;
  float acc[GM], m_run[GM], l_run[GM];
#pragma unroll
  for (int g = 0; g < GM; ++g) { acc[g] = 0.f; m_run[g] = -INFINITY; l_run[g] = 0.f; }

  const T* kp = reinterpret_cast<const T*>(a.k_pages);
  const T* vp = reinterpret_cast<const T*>(a.v_pages);
  const size_t bt_row = (size_t)b * a.max_blocks;

  for (int n0 = n_begin; n0 < n_end; n0 += kThreads) {
    // ---- phase A: one slot per thread ----
    const int n = n0 + tid;
    float s[GM];
#pragma unroll
    for (int g = 0; g < GM; ++g) s[g] = -INFINITY;
    bool take = n < n_end;
    int pos_k = n, page = 0;
    const int j = n / P, sl = n % P;
    if (take) {
      page = max(min(a.block_tables[bt_row + j], a.num_pages - 1), 0);  // a corrupt id reads a wrong page, never faults
      if (a.block_valid_mask) take = (a.block_valid_mask[bt_row + j] >> sl) & 1u;
      if (a.block_positions) pos_k = a.block_positions[bt_row + j] + sl;
      if (a.causal && pos_k > pos_q) take = false;
    }
    if (take) {
      float dot[GM];
#pragma unroll
      for (int g = 0; g < GM; ++g) dot[g] = 0.f;
      const size_t head_granules = ((size_t)page * a.Hkv + hk) * (size_t)(D / X) * P;  // in granules
      const float fpos = (float)pos_k;
      if (!a.interleaved) {
        for (int c = 0; c < half / X; ++c) {
          float x0[X], x1[X];
          load_granule<KV>(kp, head_granules + (size_t)c * P + sl, x0);
          load_granule<KV>(kp, head_granules + (size_t)(c + half / X) * P + sl, x1);
#pragma unroll
          for (int e = 0; e < X; ++e) {
            const int i = c * X + e;
            float sn, cs;
            sincospif(2.0f * turns_frac(fpos, a.freq_hi[i], a.freq_lo[i]), &sn, &cs);
            const float k0 = x0[e] * cs - x1[e] * sn, k1 = x1[e] * cs + x0[e] * sn;
            _Pragma("unroll") for (int g = 0; g < GM; ++g)
              if (g < G) dot[g] += lds.qhat[g * D + i] * k0 + lds.qhat[g * D + i + half] * k1;
          }
        }
      } else {
        for (int c = 0; c < D / X; ++c) {
          float x[X];
          load_granule<KV>(kp, head_granules + (size_t)c * P + sl, x);
#pragma unroll
          for (int e = 0; e < X; e += 2) {
            const int i = (c * X + e) / 2;
            float sn, cs;
            sincospif(2.0f * turns_frac(fpos, a.freq_hi[i], a.freq_lo[i]), &sn, &cs);
            const float k0 = x[e] * cs - x[e + 1] * sn, k1 = x[e + 1] * cs + x[e] * sn;
            _Pragma("unroll") for (int g = 0; g < GM; ++g)
              if (g < G) dot[g] += lds.qhat[g * D + 2 * i] * k0 + lds.qhat[g * D + 2 * i + 1] * k1;
          }
        }
      }
      const float ksc = KV == MEPIC_F8E4M3 ? a.k_scales[page] : 1.f;
      _Pragma("unroll") for (int g = 0; g < GM; ++g)
        if (g < G) s[g] = dot[g] * ksc;
    }

    // ---- online softmax over the tile, per head ----
    _Pragma("unroll") for (int g = 0; g < GM; ++g) {
      if (g >= G) continue;
      const float wm = wave_max(s[g]);
      if (lane == 0) lds.red[wave * GM + g] = wm;
    }
    __syncthreads();
    float alpha[GM];
    _Pragma("unroll") for (int g = 0; g < GM; ++g) {
      if (g >= G) continue;
      float tm = lds.red[g];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) tm = fmaxf(tm, lds.red[w * GM + g]);
      const float m_new = fmaxf(m_run[g], tm);
      alpha[g] = m_new == -INFINITY ? 1.f : exp2f(m_run[g] - m_new);
      m_run[g] = m_new;
      const float p = take ? exp2f(s[g] - (m_new == -INFINITY ? 0.f : m_new)) : 0.f;
      lds.sc[g * kThreads + tid] = p;
      s[g] = p;
    }
    lds.took[tid] = take ? 1 : 0;
    __syncthreads();  // red fully read, sc and took fully written
    _Pragma("unroll") for (int g = 0; g < GM; ++g) {
      if (g >= G) continue;
      const float ws = wave_sum(s[g]);
      if (lane == 0) lds.red[wave * GM + g] = ws;
    }
    __syncthreads();
    _Pragma("unroll") for (int g = 0; g < GM; ++g) {
      if (g >= G) continue;
      float ts = lds.red[g];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) ts += lds.red[w * GM + g];
      l_run[g] = l_run[g] * alpha[g] + ts;
      acc[g] *= alpha[g];
    }

    // ---- phase B: p * V. Thread owns dim d_own and blocks part, part+parts, ... of the tile ----
    const int tile_blocks = (min(n0 + kThreads, n_end) - n0 + P - 1) / P;
    for (int jb = part; jb < tile_blocks; jb += parts) {
      const int nb0 = n0 + jb * P;  // first slot of the block; n0 is a multiple of P
      const int pg = max(min(a.block_tables[bt_row + nb0 / P], a.num_pages - 1), 0);
      const float vsc = KV == MEPIC_F8E4M3 ? a.v_scales[pg] : 1.f;
      const size_t row = (((size_t)pg * a.Hkv + hk) * D + d_own) * (size_t)P;  // in elements
      for (int c = 0; c < P / X; ++c) {
        float v[X];
        load_granule<KV>(vp, row / X + c, v);
#pragma unroll
        for (int e = 0; e < X; ++e) {
          const int rel = jb * P + c * X + e;  // slot index inside the tile
          // a slot that does not take part (at or past kv_len, a pad slot the valid mask drops, a key the causal rule
          // hides) may hold anything, even NaN, and 0 x NaN is NaN: never let its V into the sum
          const float vv = lds.took[rel] ? v[e] * vsc : 0.f;
          _Pragma("unroll") for (int g = 0; g < GM; ++g)
            if (g < G) acc[g] += lds.sc[g * kThreads + rel] * vv;
        }
      }
    }
    __syncthreads();  // sc and red are rewritten by the next tile
  }

  // ---- fold the `parts` partial sums of each dim and write the split's partial result ----
  _Pragma("unroll") for (int g = 0; g < GM; ++g)
    if (g < G) lds.sc[g * kThreads + tid] = acc[g];
  __syncthreads();
  if (part == 0) {
    _Pragma("unroll") for (int g = 0; g < GM; ++g) {
      if (g >= G) continue;
      float o = 0.f;
      for (int pp = 0; pp < parts; ++pp) o += lds.sc[g * kThreads + pp * D + d_own];
      const size_t row = (size_t)t * a.Hq + (size_t)hk * a.G + g0 + g;
      if (direct) {
        const float r = l_run[g] != 0.f ? o / l_run[g] : 0.f;  // as merge_row
        if (a.q_dtype == MEPIC_F32) reinterpret_cast<float*>(a.out)[row * D + d_own] = r;
        else reinterpret_cast<uint16_t*>(a.out)[row * D + d_own] = (uint16_t)pack2_bf16(r, r);
      } else {
        const size_t pr = row * a.n_splits + split;
        a.part_o[pr * D + d_own] = o;
        if (d_own == 0) {
          a.part_ml[pr * 2] = m_run[g];
          a.part_ml[pr * 2 + 1] = l_run[g];
        }
      }
    }
  }
}

// Heads g_begin .. g_end - 1 of the KV head, four at a time (the matrix-core kernels' fallback: rare, so small rather than
// fast).
template <int KV, int kThreads>
__device__ __forceinline__ void scalar_attend_all(const AttnArgs& a, ScalarLds<4, kThreads>& lds, int t, int b, int hk,
                                                  int g_begin, int g_end, int n_begin, int n_end, int split, bool direct) {
#pragma unroll 1
  for (int g0 = g_begin; g0 < g_end; g0 += 4)
    scalar_attend<KV, 4, kThreads>(a, lds, t, b, hk, g0, min(4, g_end - g0), n_begin, n_end, split, direct);
}

}  // namespace mepic
