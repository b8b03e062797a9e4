// Merge kernel of the general path of fused-RoPE paged attention (§3.3.3): the same number of split-K partials for every
// (query token, query head).
#include "merge_partials.h"

namespace mepic {
namespace {

// Merge the per-split partials of one (query token, query head).
template <int D, typename Out, int kThreads>
__global__ __launch_bounds__(kThreads) void combine_kernel(const AttnArgs a) {
  const int row = blockIdx.x;
  merge_row<D, kThreads>(a.part_ml + (size_t)row * a.n_splits * 2, a.part_o + (size_t)row * a.n_splits * D, a.n_splits,
                         a.n_splits, reinterpret_cast<Out*>(a.out) + (size_t)row * D);
}

template <int D, typename Out>
void launch_one(const AttnArgs& a, hipStream_t s) {
  const int rows = a.n_q * a.Hq;
  if (rows <= kMergeFewRows)
    hipLaunchKernelGGL((combine_kernel<D, Out, kMergeThreadsFew>), dim3(rows), dim3(kMergeThreadsFew), 0, s, a);
  else
    hipLaunchKernelGGL((combine_kernel<D, Out, kMergeThreads>), dim3(rows), dim3(kMergeThreads), 0, s, a);
}

}  // namespace

hipError_t launch_combine(const AttnArgs& a, hipStream_t s) {
  const bool f32 = a.q_dtype == MEPIC_F32;
  if (a.D == 128 && f32) launch_one<128, float>(a, s);
  else if (a.D == 128) launch_one<128, uint16_t>(a, s);
  else if (f32) launch_one<64, float>(a, s);
  else launch_one<64, uint16_t>(a, s);
  return hipGetLastError();
}

}  // namespace mepic
