// General-path kernel of fused-RoPE paged attention (§3.3.3) for fp32 pages, and the split-K combine kernel.
//
// Handles both rotary pairings, decode and causal prefill, the optional per-block positions and valid masks. One
// workgroup of 256 threads serves one (query token, KV head, split) with the scalar body of attn_scalar.h: the G query
// heads that share the KV head reuse every rotated key. Partial (max, sum, un-normalised output) per split go to the
// workspace; combine_kernel merges them.
#include "attn_scalar.h"
#include "merge_partials.h"

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

// Merge the per-split partials of one (query token, query head).
template <int D, typename Out>
__global__ __launch_bounds__(kMergeThreads) void combine_kernel(const AttnArgs a) {
  const int row = blockIdx.x;
  merge_row<D>(a.part_ml + (size_t)row * a.n_splits * 2, a.part_o + (size_t)row * a.n_splits * D, a.n_splits, a.n_splits,
               reinterpret_cast<Out*>(a.out) + (size_t)row * D);
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
  const dim3 grid(a.n_q * a.Hq), block(kMergeThreads);
  const bool f32 = a.q_dtype == MEPIC_F32;
  if (a.D == 128 && f32) hipLaunchKernelGGL((combine_kernel<128, float>), grid, block, 0, s, a);
  else if (a.D == 128) hipLaunchKernelGGL((combine_kernel<128, uint16_t>), grid, block, 0, s, a);
  else if (f32) hipLaunchKernelGGL((combine_kernel<64, float>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((combine_kernel<64, uint16_t>), grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace mepic
