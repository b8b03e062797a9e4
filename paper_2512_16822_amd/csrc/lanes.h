// What the matrix-core kernels share: operand fragments, wave-uniform values and reads, exchanges between lanes.
#pragma once
#include "attn_common.h"

namespace mepic {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

union Frag {  // one 16-byte operand fragment
  uint4 u;
  bf16x8 v;
  f16x8 hv;
  uint32_t w[4];
};

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Wave-uniform read of a read-only int32 input through the scalar unit (s_load): unlike a vector load it
// does not share the vector-memory counter, so waiting for it never drains the K/V loads in flight.
typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;
__device__ __forceinline__ int sload(const int32_t* p, size_t idx) {
  return ((const_i32_ptr)(uintptr_t)p)[idx];
}

// Two waves share a SIMD here, and the one that came first gets every issue slot that both want: with equal parts of the work it is done
// first, and the other goes on alone with nothing to fill its waits. So the later one is preferred in five of every eight turns, which the
// caller counts through the wave's work: of 128 requests of 2 - 33 K e4m3 slots, plain decode, the first waves end after 132 us and the
// others after 177; so preferred all after 159 - 169, and the call takes 174 us, not 181. 64 requests of 4.3 K bf16 slots 70.6 -> 69.2, with
// masks 84.0 -> 80.2; 16 of 2.2 K behind a commit 21.4 -> 21.2. (Half and three quarters of the turns, by ones, gain 1 - 2 % less; a
// preference in all of many turns turns the sides round. Progress compared through LDS ends them together too, but in step with each
// other: nothing gained, 0.9 us lost on the last.) A wave of up to five turns is preferred in all of them, which in plain decode is
// worth as much: us a call without and with, 100 requests of 0.3 - 1 K bf16 slots 24.95 and 24.2, e4m3 20.6 and 20.3, 30 of 0.5 - 1 K e4m3 slots
// 14.35 and 13.8; the most it cost there is 1 % (128 of 0.3 - 1 K on 4 KV heads 21.8 and 22.0). Counted afresh for every run, though, waves of
// several short runs had it throughout: 500 requests of 100 - 300 slots 59.05, without turns 58.4, counted through 57.9.
// (s_setprio takes constants only. The branch between two is out of the compiler's sight: as one of its own it cost general decode calls
// of few steps 0.2 us, taken or not.)
__device__ __forceinline__ void take_turns(bool later, int turn) {
  const int first = uni(later && (turn & 7) < 5);
  asm volatile("s_cmp_lg_u32 %0, 0\n\ts_cbranch_scc0 1f\n\ts_setprio 1\n\ts_branch 2f\n1:\n\ts_setprio 0\n2:" ::"s"(first) : "scc");
}

// The value of the lane kBy places up in the row of 16 lanes (0 past its end).
template <int kBy>
__device__ __forceinline__ float lane_up(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x100 + kBy, 0xf, 0xf, true));
}

// Maximum over the four lanes l, l^16, l^32, l^48 (the four k-groups of one head), in every lane.
__device__ __forceinline__ float max_over_kgroups(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const uint32_t v = __float_as_uint(y);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float sum_over_kgroups(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const uint32_t v = __float_as_uint(y);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

}  // namespace mepic
