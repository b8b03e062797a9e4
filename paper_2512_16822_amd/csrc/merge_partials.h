// Merge of split-K partials: one workgroup of kThreads (64 to 256) threads per (query token, query head). Partial s holds a
// reference maximum (log2 units), a sum and an un-normalised row of D fp32 values; with m* the largest maximum,
//   out = sum_s 2^(m_s - m*) o_s / sum_s 2^(m_s - m*) l_s          (all zeros when no slot took part).
// A partial no slot took part in has maximum -inf and sum 0; its row may hold anything and is left out. Every other one counts,
// however small its weight, so that a NaN or Inf of its row or its sum is in the result wherever the context was cut.
//
// What a merge of tens of partials costs is memory latency, not bytes, so there is as little as possible in its chain of dependent loads:
// lane i of every wave takes the maximum and the sum of partial i (64 at a time, one coalesced load), and each thread's first row is
// requested before the number of partials is known. Groups of D / 4 threads take every kGroups-th partial, a thread four dims of it; LDS
// adds the groups up. With 256 threads all other rows of up to 64 partials are requested as soon as their number is known (two at a
// time, one turn ahead, were four trips to memory where there are 54; all of them before it is known reads what nobody wrote: a commit and
// 16 requests of 2.2 K slots 21.2 -> 22.1 us). us a call before and after: 4 requests of 1.7 K slots, 54 partials a row, 12.4 -> 11.75, that
// commit and 16 requests, 16 partials, 21.2 -> 20.95, 2 planned requests of 7 K 19.7 -> 17.3.
#pragma once
#include "attn_common.h"

namespace mepic {

template <typename Out> __device__ __forceinline__ void store4(Out* dst, const float4& v);
template <> __device__ __forceinline__ void store4<float>(float* dst, const float4& v) { *reinterpret_cast<float4*>(dst) = v; }
template <> __device__ __forceinline__ void store4<uint16_t>(uint16_t* dst, const float4& v) {
  uint2 p;
  p.x = pack2_bf16(v.x, v.y);
  p.y = pack2_bf16(v.z, v.w);
  *reinterpret_cast<uint2*>(dst) = p;
}

// Reductions over the wave without LDS: rotations inside rows of 16 lanes, then the two lane-swap instructions.
template <int kRor>
__device__ __forceinline__ float row_ror(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x120 + kRor, 0xf, 0xf, true));
}
template <typename Op>
__device__ __forceinline__ float wave_reduce(float x, Op op) {
  x = op(x, row_ror<1>(x));
  x = op(x, row_ror<2>(x));
  x = op(x, row_ror<4>(x));
  x = op(x, row_ror<8>(x));
  uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  x = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
  u = __float_as_uint(x);
  const auto b = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return op(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Threads per row. Up to four rows per compute unit leave it nearly idle: 256 threads (us a call with 128 and 256: 528 rows of a plan 17.3
// and 16.8, 624 20.3 and 19.8, 864 31.1 and 30.9; general decode of 500 - 1000 rows even). With more rows there are enough loads in
// flight, and the extra waves cost: 2048 batched rows 55.3 and 55.7, 2048 plain ones 69.4 and 70.1. 512 threads: 0.1 - 0.2 us more for few
// partials, 0.1 less for 54.
constexpr int kMergeThreads = 128, kMergeThreadsFew = 256, kMergeFewRows = 1024;

// ml: [room][2], po: [room][D], out: the row; ns <= room partials exist (room is known before ns has been loaded, so the
// first loads go by room).
template <int D, int kThreads, typename Out>
__device__ __forceinline__ void merge_row(const float* ml, const float* po, int room, int ns, Out* out) {
  constexpr int kCols = D / 4, kGroups = kThreads / kCols;
  constexpr bool kAll = kThreads == kMergeThreadsFew;  // the rows of 64 partials at once
  constexpr int kAhead = kAll ? 64 / kGroups : 2;
  static_assert(kThreads % kCols == 0 && 64 % kGroups == 0, "the groups take the 64 partials of a turn in whole rounds");
  __shared__ float4 num_s[kGroups][kCols];
  const int lane = threadIdx.x & 63, part = threadIdx.x / kCols, dq = threadIdx.x % kCols;
  const float2* ml2 = reinterpret_cast<const float2*>(ml);
  const float4* po4 = reinterpret_cast<const float4*>(po) + dq;
  float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
  float den = 0.f, m = -INFINITY;
  auto row = [&](int s) { return s < ns ? po4[(size_t)s * kCols] : make_float4(0.f, 0.f, 0.f, 0.f); };
  auto add = [&](const float4& x, float w) {
    if (!(w < 0.f)) {  // (a weight may be NaN)
      num.x += w * x.x; num.y += w * x.y; num.z += w * x.z; num.w += w * x.w;
    }
  };
  float2 e = lane < room ? ml2[lane] : make_float2(-INFINITY, 0.f);
  float4 x[kAhead];
  x[0] = part < room ? po4[(size_t)part * kCols] : make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s0 = 0; s0 < ns; s0 += 64) {  // (one turn but for the longest contexts)
    int s = s0 + part;
    if (s0 > 0) {
      e = ml2[min(s0 + lane, ns - 1)];
      x[0] = row(s);
    }
#pragma unroll
    for (int i = 1; i < kAhead; ++i)
      if (!kAll || s0 + i * kGroups < ns) x[i] = row(s + i * kGroups);
    if (s0 + lane >= ns) e = make_float2(-INFINITY, 0.f);
    const bool took = e.x != -INFINITY || e.y != 0.f;
    const int s_end = min(ns, s0 + 64);
    const float m_new = fmaxf(m, wave_reduce(e.x, [](float x, float y) { return fmaxf(x, y); }));
    if (m_new != m && m != -INFINITY) {
      const float f = __builtin_amdgcn_exp2f(m - m_new);
      num.x *= f; num.y *= f; num.z *= f; num.w *= f;
      den *= f;
    }
    m = m_new;
    const float w = took ? __builtin_amdgcn_exp2f(e.x - m) : -1.f;  // (NaN where all scores of the row are)
    den += wave_reduce(took ? w * e.y : 0.f, [](float x, float y) { return x + y; });
    // (every lane runs as many turns as the first group: the shuffles need all of them)
    if constexpr (kAll) {
#pragma unroll
      for (int i = 0; i < kAhead; ++i)
        if (s0 + i * kGroups < ns) add(x[i], __shfl(w, part + i * kGroups));
    } else {
      for (int i = s0; i < s_end; i += 2 * kGroups, s += 2 * kGroups) {
        const float4 u = x[0], v = x[1];
        x[0] = row(s + 2 * kGroups);
        x[1] = row(s + 3 * kGroups);
        add(u, __shfl(w, (s - s0) & 63));
        add(v, __shfl(w, (s + kGroups - s0) & 63));
      }
    }
  }
  num_s[part][dq] = num;
  __syncthreads();
  if (part == 0) {
#pragma unroll
    for (int p = 1; p < kGroups; ++p) {
      const float4 x = num_s[p][dq];
      num.x += x.x; num.y += x.y; num.z += x.z; num.w += x.w;
    }
    const float inv = 1.f / den;
    store4<Out>(out + 4 * dq, den != 0.f ? make_float4(num.x * inv, num.y * inv, num.z * inv, num.w * inv)
                                         : make_float4(0.f, 0.f, 0.f, 0.f));
  }
}

}  // namespace mepic
