// Merge kernel of the general path of fused-RoPE paged attention (§3.3.3): the same number of split-K partials for every
// (query token, query head).
#include "merge_partials.h"

namespace mepic {
namespace {

// Merge the per-split partials of one (query token, query head).
template <int D, typename Out>
__global__ __launch_bounds__(kMergeThreads) void combine_kernel(const AttnArgs a) {
  const int row = blockIdx.x;
  merge_row<D>(a.part_ml + (size_t)row * a.n_splits * 2, a.part_o + (size_t)row * a.n_splits * D, a.n_splits, a.n_splits,
               reinterpret_cast<Out*>(a.out) + (size_t)row * D);
}

}  // namespace

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
