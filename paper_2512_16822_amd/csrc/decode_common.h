// What the plain and the batched decode kernel share: page ids, page loads, and the two-term dot products that rotate bf16 keys.
#pragma once
#include <type_traits>

#include "lanes.h"

namespace mepic {

// Two fp32 -> packed fp16 pair, round to nearest even.
__device__ __forceinline__ uint32_t pack_f16x2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
}

// A page id as the kernels use it: forced into [0, num_pages) so that a corrupt block table reads a wrong page
// instead of faulting (the result of that request is then unspecified, nothing else is affected).
__device__ __forceinline__ int safe_page(int id, int num_pages) { return max(min(id, num_pages - 1), 0); }

// 16- and 8-byte loads of page data, optionally with the non-temporal hint (the line is not kept in the caches):
// right when every page is read by one request only, wrong when pages are shared between requests.
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
template <bool kNT>
__device__ __forceinline__ uint4 load_page(const uint4* p) {
  if constexpr (kNT) {
    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    return make_uint4(v[0], v[1], v[2], v[3]);
  } else {
    return *p;
  }
}
template <bool kNT>
__device__ __forceinline__ uint2 load_page(const uint2* p) {
  if constexpr (kNT) {
    const u32x2_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x2_t*>(p));
    return make_uint2(v[0], v[1]);
  } else {
    return *p;
  }
}

// Eight two-term dot products on packed bf16 words, fp32 results: l_i = e_i . ca_i, h_i = e_i . cb_i, where
// e_i = (low element, high element) of a rotary pair and ca = (cos, -sin), cb = (sin, cos) as packed bf16.
// One block of eight v_dot2_f32_bf16 closed by four wait states: another vector instruction may neither read the
// result of a dot instruction for three wait states nor rewrite its register for four, and the compiler places those
// only around its own builtin. Within the block no dot reads or rewrites another's result; the outputs are
// early-clobber, so none shares a register with an input. Validated on ROCm 7.2 (AMD clang 22, gfx950); the
// library's self-test entry point runs this block alone against fp32 arithmetic so that a toolchain that breaks the
// rule shows up as a failed test and not as slightly wrong attention.
__device__ __forceinline__ void dot_rotate_block(uint32_t e0, uint32_t e1, uint32_t e2, uint32_t e3, uint32_t ca0,
                                                 uint32_t cb0, uint32_t ca1, uint32_t cb1, uint32_t ca2, uint32_t cb2,
                                                 uint32_t ca3, uint32_t cb3, float& l0, float& l1, float& l2, float& l3,
                                                 float& h0, float& h1, float& h2, float& h3) {
  asm("v_dot2_f32_bf16 %0, %8, %12, 0\n\t"
      "v_dot2_f32_bf16 %1, %9, %14, 0\n\t"
      "v_dot2_f32_bf16 %2, %10, %16, 0\n\t"
      "v_dot2_f32_bf16 %3, %11, %18, 0\n\t"
      "v_dot2_f32_bf16 %4, %8, %13, 0\n\t"
      "v_dot2_f32_bf16 %5, %9, %15, 0\n\t"
      "v_dot2_f32_bf16 %6, %10, %17, 0\n\t"
      "v_dot2_f32_bf16 %7, %11, %19, 0\n\t"
      "s_nop 3"
      : "=&v"(l0), "=&v"(l1), "=&v"(l2), "=&v"(l3), "=&v"(h0), "=&v"(h1), "=&v"(h2), "=&v"(h3)
      : "v"(e0), "v"(e1), "v"(e2), "v"(e3), "v"(ca0), "v"(cb0), "v"(ca1), "v"(cb1), "v"(ca2), "v"(cb2), "v"(ca3),
        "v"(cb3));
}

}  // namespace mepic
