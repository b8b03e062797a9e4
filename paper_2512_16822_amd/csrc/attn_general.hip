// General-path kernel of fused-RoPE paged attention (§3.3.3) for fp32 pages, and the split-K combine kernel.
//
// Handles both rotary pairings, decode and causal prefill, the optional per-block positions and valid masks. One
// workgroup of 256 threads serves one (query token, KV head, split) with the scalar body of attn_scalar.h: the G query
// heads that share the KV head reuse every rotated key. Partial (max, sum, un-normalised output) per split go to the
// workspace; combine_kernel merges them.
#include "attn_scalar.h"

namespace mepic {
namespace {

constexpr int kThreads = 256;

template <int GM>
__global__ __launch_bounds__(kThreads) void attn_general_kernel(const AttnArgs a) {
  const int tid = threadIdx.x;
  const int t = blockIdx.x, hk = blockIdx.y, split = blockIdx.z;
  __shared__ ScalarLds<GM, kThreads> lds;
  __shared__ int s_req;

  // which request owns this query token
  if (tid == 0) {
    int b = t;
    if (a.cu_q_lens) {
      int lo = 0, hi = a.B - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.cu_q_lens[mid] <= t) lo = mid; else hi = mid - 1;
      }
      b = lo;
    }
    s_req = b;
  }
  __syncthreads();
  const int b = s_req;
  const int L = a.kv_lens[b];
  const int n_begin = split * a.blocks_per_split * a.P;
  const int n_end = min(L, (split + 1) * a.blocks_per_split * a.P);
  scalar_attend<MEPIC_F32, GM, kThreads>(a, lds, t, b, hk, 0, a.G, n_begin, n_end, split, false);
}

// Merge the per-split partials of one (query token, query head): with m* the largest split maximum,
// out = sum_s 2^(m_s - m*) o_s / sum_s 2^(m_s - m*) l_s (all zeros when no slot took part).
__global__ __launch_bounds__(128) void combine_kernel(const AttnArgs a) {
  const int row = blockIdx.x, d = threadIdx.x;
  if (d >= a.D) return;
  const float* ml = a.part_ml + (size_t)row * a.n_splits * 2;
  const float* po = a.part_o + (size_t)row * a.n_splits * a.D;
  float m = -INFINITY;
  for (int s = 0; s < a.n_splits; ++s) m = fmaxf(m, ml[2 * s]);
  float num = 0.f, den = 0.f;
  if (m != -INFINITY) {
    for (int s = 0; s < a.n_splits; ++s) {
      const float ms = ml[2 * s];
      if (ms == -INFINITY) continue;
      const float w = exp2f(ms - m);
      num += w * po[(size_t)s * a.D + d];
      den += w * ml[2 * s + 1];
    }
  }
  const float o = den > 0.f ? num / den : 0.f;
  const size_t idx = (size_t)row * a.D + d;
  if (a.q_dtype == MEPIC_F32) reinterpret_cast<float*>(a.out)[idx] = o;
  else reinterpret_cast<uint16_t*>(a.out)[idx] = (uint16_t)f32_to_bf16_bits(o);
}

}  // namespace

hipError_t launch_general(const AttnArgs& a, hipStream_t s) {
  const dim3 grid(a.n_q, a.Hkv, a.n_splits), block(kThreads);
  if (a.G <= 1) hipLaunchKernelGGL((attn_general_kernel<1>), grid, block, 0, s, a);
  else if (a.G <= 2) hipLaunchKernelGGL((attn_general_kernel<2>), grid, block, 0, s, a);
  else if (a.G <= 4) hipLaunchKernelGGL((attn_general_kernel<4>), grid, block, 0, s, a);
  else if (a.G <= 8) hipLaunchKernelGGL((attn_general_kernel<8>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((attn_general_kernel<16>), grid, block, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_combine(const AttnArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(combine_kernel, dim3(a.n_q * a.Hq), dim3(128), 0, s, a);
  return hipGetLastError();
}

}  // namespace mepic
