// What the restoration kernels share on the device: vector types, bf16 rounding of a pair, the rotation of a
// pair, and the lookup of a token row's position and context.
#pragma once

#include <type_traits>
#include <utility>

#include "hcache_internal.h"

namespace hc {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));   // round to nearest even
}

// Rotation of a RoPE pair (a, b) by (cos, sin).  The roundings are spelt out: kernels that promise the same bits may
// not leave it to the compiler which of the two products is fused.
__device__ __forceinline__ void rotate_pair(float& a, float& b, float c, float s) {
  const float ra = __builtin_fmaf(a, c, -(b * s));
  b = __builtin_fmaf(b, c, a * s);
  a = ra;
}

// f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>)
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) { static_for_impl(f, std::make_integer_sequence<int, N>{}); }

// Position and context of token row t (of a batch without positions, every context starts at pos_base).
__device__ __forceinline__ void token_place(const RestoreArgs& a, int t, int& pos, int& seq) {
  pos = a.positions ? a.positions[t] : a.pos_base + t;
  if (a.cu_seqlens) {                                     // largest s with cu[s] <= t
    int lo = 0, hi = a.n_seq;                             // invariant: cu[lo] <= t < cu[hi]
    int first = a.cu_seqlens[0];                          // first row of context lo
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      const int c = a.cu_seqlens[mid];
      if (c <= t) { lo = mid; first = c; } else hi = mid;
    }
    seq = lo;
    if (!a.positions) pos = a.pos_base + t - first;
  }
}

}  // namespace hc
