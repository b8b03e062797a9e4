// Shared device helpers of the general path's matrix-core kernels (attn_prefill_split.hip, attn_decode_split.hip).
//
// "Split" precision: an fp32 value x enters a bf16 matrix product as two operands, hi = bf16(x) and lo = bf16(x - hi),
// which together carry 16 significant bits (relative error 2^-18). A product of two such values is three matrix
// products (hi hi + hi lo + lo hi; the dropped lo lo is of the size of the error), a product with an operand that bf16
// holds exactly (stored bf16 values, e4m3 codes) two. Everything else - phases, rotation, softmax, sums - is fp32.
//
// That is less than the 24 bits of fp32 operands. A score is off by at most 2^-15 x scale x sum |q_i k_i| (two operands and the
// dropped product 2^-18 each, 128 fp32 sums 2^-17, the sines 2^-19), however much of the sum cancels. On values of unit variance,
// and on keys with a common offset per dim of eight times their spread (scale x sum |q_i k_i| up to 750), what is left is the
// output's own rounding to bf16: 1.3e-3 to 1.7e-3 of the norm, and beyond that rounding 1.2e-4 of the largest output at most.
#pragma once
#include <atomic>

#include "lanes.h"

namespace mepic {

// Ask for more dynamic LDS than a kernel gets by default: once per kernel and device (the attribute sticks to a device's
// copy of the kernel). `asked` is the kernel's own, one bit for each device.
inline hipError_t allow_lds(const void* kernel, size_t bytes, std::atomic<uint64_t>& asked) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;
  if (asked.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) asked.fetch_or(bit, std::memory_order_release);
  return e;
}

// Two fp32 values -> their packed bf16 heads and packed bf16 remainders. (x - head as a two-term dot product of the packed
// word with (-1, 0) saves two of the six instructions and measured no faster here and 5 % slower in the prefill kernel.)
__device__ __forceinline__ void split2(float x0, float x1, uint32_t& hi, uint32_t& lo) {
  hi = pack2_bf16(x0, x1);
  lo = pack2_bf16(x0 - __uint_as_float(hi << 16), x1 - __uint_as_float(hi & 0xffff0000u));
}

__device__ __forceinline__ float uni_f(float v) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v))); }

// Eight stored elements (one granule of bf16, or half a granule of e4m3 codes) as loaded.
template <bool kFp8> struct Raw8;
template <> struct Raw8<false> { uint4 r; };
template <> struct Raw8<true> { uint2 r; };

template <bool kFp8>
__device__ __forceinline__ void widen8(const Raw8<kFp8>& in, float (&x)[8]) {
  if constexpr (kFp8) {
    const uint32_t w[2] = {in.r.x, in.r.y};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const f32x2 a = __builtin_amdgcn_cvt_pk_f32_fp8(w[i], false), b = __builtin_amdgcn_cvt_pk_f32_fp8(w[i], true);
      x[4 * i] = a[0]; x[4 * i + 1] = a[1]; x[4 * i + 2] = b[0]; x[4 * i + 3] = b[1];
    }
  } else {
    const uint32_t w[4] = {in.r.x, in.r.y, in.r.z, in.r.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = __uint_as_float(w[i] << 16);
      x[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
}

// Eight stored elements as packed bf16 (exact for e4m3 codes, whose page scale is applied elsewhere).
template <bool kFp8>
__device__ __forceinline__ Frag bf16_of8(const Raw8<kFp8>& in) {
  Frag f;
  if constexpr (kFp8) {
    const uint32_t w[2] = {in.r.x, in.r.y};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const f32x2 a = __builtin_amdgcn_cvt_pk_f32_fp8(w[i], false), b = __builtin_amdgcn_cvt_pk_f32_fp8(w[i], true);
      f.w[2 * i] = __builtin_amdgcn_perm(__float_as_uint(a[1]), __float_as_uint(a[0]), 0x07060302u);
      f.w[2 * i + 1] = __builtin_amdgcn_perm(__float_as_uint(b[1]), __float_as_uint(b[0]), 0x07060302u);
    }
  } else {
    f.u = in.r;
  }
  return f;
}

// Keep the elements of `f` whose bit of `keep` (8 bits) is set, zero the others.
__device__ __forceinline__ void mask8(Frag& f, uint32_t keep) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
    f.w[i] &= ((keep >> (2 * i)) & 1u ? 0x0000ffffu : 0u) | ((keep >> (2 * i + 1)) & 1u ? 0xffff0000u : 0u);
}

}  // namespace mepic
