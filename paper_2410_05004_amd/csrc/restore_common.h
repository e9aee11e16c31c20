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

// What is left of a wave's tile of one 64-row pair group (K or V) x 16 NB tokens once the sums are known: scale, rotate, round and
// store, everything per token in the lane that owns it.  acc[i][j]: 16-row block i, token block j; row[j]: pool row of the token's K, or -1;
// nmu: -mean / std (LayerNorm only); dst0: where row 0 has the lane's first feature; aff: (S, C) of its first row; load_cs(j, cs): (cos, sin) of its eight
// pairs for the token of block j, asked for a block ahead.
template <int NB, bool LN, bool AFF, bool ROT, class LoadCs>
__device__ __forceinline__ void finish_blocks(const RestoreArgs& a, const f32x4 (&acc)[4][NB], const int (&row)[NB], const float (&rstd)[NB],
                                              const float (&nmu)[NB], const float2* aff, uint16_t* dst0, LoadCs&& load_cs) {
  const int style = a.rope_style, half = a.head_dim >> 1;
  float4 sc[4][2];
  if constexpr (AFF) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sc[i][0] = *reinterpret_cast<const float4*>(aff + 16 * i);
      sc[i][1] = *reinterpret_cast<const float4*>(aff + 16 * i + 2);
    }
  }
  float4 cs[2][4];
  if constexpr (ROT) load_cs(0, cs[0]);
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    if constexpr (ROT) { if (j + 1 < NB) load_cs(j + 1, cs[(j + 1) & 1]); }
    auto val2 = [&](int i, int v, float& y0, float& y1) __attribute__((always_inline)) {
      if constexpr (!AFF) {
        y0 = acc[i][j][v] * rstd[j];
        y1 = acc[i][j][v + 1] * rstd[j];
      } else {
        const float4 s4 = sc[i][v >> 1];
        const float c0 = LN ? __builtin_fmaf(nmu[j], s4.x, s4.y) : s4.y;
        const float c1 = LN ? __builtin_fmaf(nmu[j], s4.z, s4.w) : s4.w;
        y0 = __builtin_fmaf(acc[i][j][v], rstd[j], c0);
        y1 = __builtin_fmaf(acc[i][j][v + 1], rstd[j], c1);
      }
    };
    float fa[8], fb[8];                                   // first and second members of the lane's eight pairs
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      float a0, a1, b0, b1;
      val2(e >> 2, e & 3, a0, a1);
      val2(2 + (e >> 2), e & 3, b0, b1);
      if constexpr (ROT) {
        const float4 c4 = cs[j & 1][e >> 1];
        rotate_pair(a0, b0, c4.x, c4.y);
        rotate_pair(a1, b1, c4.z, c4.w);
      }
      fa[e] = a0; fa[e + 1] = a1;
      fb[e] = b0; fb[e + 1] = b1;
    }
    u32x4 w0, w1;
    if (style == 1) {
      w0 = u32x4{pack2(fa[0], fb[0]), pack2(fa[1], fb[1]), pack2(fa[2], fb[2]), pack2(fa[3], fb[3])};
      w1 = u32x4{pack2(fa[4], fb[4]), pack2(fa[5], fb[5]), pack2(fa[6], fb[6]), pack2(fa[7], fb[7])};
    } else {
      w0 = u32x4{pack2(fa[0], fa[1]), pack2(fa[2], fa[3]), pack2(fa[4], fa[5]), pack2(fa[6], fa[7])};
      w1 = u32x4{pack2(fb[0], fb[1]), pack2(fb[2], fb[3]), pack2(fb[4], fb[5]), pack2(fb[6], fb[7])};
    }
    if (row[j] >= 0) {
      uint16_t* dst = dst0 + (size_t)row[j] * a.d_kv;
      *reinterpret_cast<u32x4*>(dst) = w0;
      *reinterpret_cast<u32x4*>(dst + (style == 1 ? 8 : half)) = w1;
    }
  }
}

}  // namespace hc
