// Float32 products on the float16 matrix cores.
//
// v_mfma_f32_16x16x4_f32 takes 32 cycles for 1024 multiply-adds, v_mfma_f32_16x16x32_f16 takes 16 for 8192 (measured 32.0 and
// 17.0, dependent or not).  A float32 operand is split into two float16 terms, x s = h + l with h = f16(x s) and
// l = f16(x s - h), and a product is l h' + h l' + h h': 3 instructions of 16 cycles where 8 of 32 stood.  h carries 11
// significant bits and l, signed, 11 more: 23 with the sign of l, of float32's 24, so an operand is off by 2^-23 of x at most, and l l' is
// left out, 2^-22 of the product at most and 2^-24 as a rule.  Against that the matrix core rounds less often than after every product, as
// the float32 instruction does.  Measured against float64
// (rms of the error over the rms of the product, normal operands): K = 32 0.88e-7 (float32 instruction 1.03e-7), K = 64 1.07e-7
// (1.45e-7), K = 128 1.38e-7 (2.02e-7): the split is the more accurate of the two.
//
// s is a power of two, so that scaling is exact: the largest entry of the columns a wavefront owns goes to [2^14, 2^15).  What is
// 2^15 times smaller than that begins to lose bits of l, which by then are 2^-40 of the largest entry: operands have to be written in
// units in which entries that matter are not much smaller (ttc_columns.hpp and ttc_squaring.hpp see to it).
#pragma once
#include "ttc_device.hpp"

namespace ttc {

typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));

// The pair in LDS with the notes of split products behind it: a type that carries its size, so that a pair without room for the
// notes does not compile.
template <int D>
using Pair = float[Cfg<D>::PAIR];

// A matrix by columns (ttc_columns.hpp) in split form: m[2q][k] and m[2q + 1][k], a lane's eight values of 32 rows, are one
// B operand of the matrix core, which visits the contraction index as k = 32 q + 16 (j / 4) + 4 g + j % 4.
template <int D, int CT>
struct SplitCols {
  halfx8 h[D / 32][CT], l[D / 32][CT];
  float inv;  // 1 / s, the same in all lanes
};

// 1 / s for the largest magnitude of a wavefront (float bits), and s from that.  The exponent is kept where both are normal.
__device__ __forceinline__ float split_unscale(uint32_t max_bits) {
  int e = (int)(max_bits >> 23);
  e = e < 15 ? 15 : (e > 254 ? 254 : e);
  return __uint_as_float((uint32_t)(e - 14) << 23);
}

__device__ __forceinline__ void split_pair(float x, float y, float s, halfx2& h, halfx2& l) {
  h = __builtin_convertvector(floatx2{x * s, y * s}, halfx2);
  l[0] = (_Float16)__builtin_fmaf(x, s, -(float)h[0]);
  l[1] = (_Float16)__builtin_fmaf(y, s, -(float)h[1]);
}

// the power of two 1 / x
__device__ __forceinline__ float power_inverse(float x) { return __uint_as_float((254u << 23) - __float_as_uint(x)); }

template <int D, int CT>
__device__ __forceinline__ void split_cols(const floatx4 (&m)[D / 16][CT], SplitCols<D, CT>& sp) {
  float big = 0.f;
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int k = 0; k < CT; ++k)
#pragma unroll
      for (int v = 0; v < 4; v += 2) {
        const float x = __builtin_fabsf(m[r][k][v]), y = __builtin_fabsf(m[r][k][v + 1]);
        // At d = 128 the IEEE maximum (NaN on top), two entries an instruction: the other one first makes quiet NaNs of signalling ones, 28
        // instructions for 16 entries (squaring T = 16, 8192 problems 10.06 -> 9.64 ms, bfloat16 T = 32, 4096 problems 5.89 -> 5.69); at
        // d = 64 registers fall out worse with it (T = 64, 4099 problems 0.900 -> 0.922).
        if constexpr (D == 128) big = __builtin_elementwise_maximum(__builtin_elementwise_maximum(big, x), y);
        else big = __builtin_fmaxf(big, __builtin_fmaxf(x, y));
      }
  sp.inv = split_unscale(wave_max_u32(__float_as_uint(big)));
  const float s = power_inverse(sp.inv);
#pragma unroll
  for (int q = 0; q < D / 32; ++q)
#pragma unroll
    for (int k = 0; k < CT; ++k)
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        const floatx4& t = m[2 * q + j / 4][k];
        halfx2 h, l;
        split_pair(t[j % 4], t[j % 4 + 1], s, h, l);
        sp.h[q][k][j] = h[0];
        sp.h[q][k][j + 1] = h[1];
        sp.l[q][k][j] = l[0];
        sp.l[q][k][j + 1] = l[1];
      }
}

// Behind the pair: four times d floats for the caller (units of the states, of the controls and of the columns of A, and the signs of A's
// diagonal), then 1 / s of every wavefront's rows of the left operand in either half.
template <int D>
__device__ __forceinline__ float* state_units(Pair<D>& W) { return W + D * Cfg<D>::PITCH; }
template <int D>
__device__ __forceinline__ float* control_units(Pair<D>& W) { return W + D * Cfg<D>::PITCH + D; }
template <int D>
__device__ __forceinline__ float* column_units(Pair<D>& W) { return W + D * Cfg<D>::PITCH + 2 * D; }
template <int D>
__device__ __forceinline__ float* diagonal_signs(Pair<D>& W) { return W + D * Cfg<D>::PITCH + 3 * D; }
template <int D>
__device__ __forceinline__ float* split_notes(Pair<D>& W, int half) { return W + D * Cfg<D>::PITCH + 4 * D + 8 * half; }

// The transpose to LDS as a left operand, into the half of the pair that begins at L: row 16 RB w + .. of the transpose is a
// column of the matrix, h in the first half of the row's d floats and l in the second, the contraction index in the matrix
// core's order.  1 / s of the wavefront's rows goes behind the pair.
template <int D>
__device__ __forceinline__ void store_split_T(Pair<D>& W, int half, const SplitCols<D, Cfg<D>::RB>& sp, int w, int i,
                                              int g) {
  using C = Cfg<D>;
  float* const o = W + half * D + (16 * C::RB * w + i) * C::PITCH + 4 * g;
#pragma unroll
  for (int k = 0; k < C::RB; ++k)
#pragma unroll
    for (int q = 0; q < D / 32; ++q) {
      *reinterpret_cast<halfx8*>(o + 16 * k * C::PITCH + 16 * q) = sp.h[q][k];
      *reinterpret_cast<halfx8*>(o + 16 * k * C::PITCH + D / 2 + 16 * q) = sp.l[q][k];
    }
  if (i == 0 && g == 0) split_notes<D>(W, half)[w] = sp.inv;
}

// and back, by the wavefront that stored it
template <int D>
__device__ __forceinline__ void read_split(const Pair<D>& W, int half, SplitCols<D, Cfg<D>::RB>& sp, int w, int i, int g) {
  using C = Cfg<D>;
  const float* const o = W + half * D + (16 * C::RB * w + i) * C::PITCH + 4 * g;
#pragma unroll
  for (int k = 0; k < C::RB; ++k)
#pragma unroll
    for (int q = 0; q < D / 32; ++q) {
      sp.h[q][k] = *reinterpret_cast<const halfx8*>(o + 16 * k * C::PITCH + 16 * q);
      sp.l[q][k] = *reinterpret_cast<const halfx8*>(o + 16 * k * C::PITCH + D / 2 + 16 * q);
    }
}

// acc = L b, or acc += SIGN L b (ADD): L a left operand in LDS as store_split_T leaves it, b by columns in split form.  A
// 16 x 16 tile is formed from zero and then scaled back into acc, under the next tile's matrix instructions.  The left operands
// of the next two k-steps are in flight while one is used; scheduling barriers keep the compiler from hoisting more.
template <int D, int CT, bool ADD = false, int SIGN = 1>
__device__ __forceinline__ void gemm_split(floatx4 (&acc)[D / 16][CT], Pair<D>& W, int half,
                                           const SplitCols<D, CT>& b, int i, int g) {
  using C = Cfg<D>;
  constexpr int NT = C::NT, NQ = D / 32, NX = NT * NQ, AHEAD = NX < 3 ? NX - 1 : 2;
  constexpr int RSEG = 65000 / (16 * C::PITCH * 4) > 0 ? 65000 / (16 * C::PITCH * 4) : 1;  // as in gemm_cols
  const float* const base = W + half * D + i * C::PITCH + 4 * g;
  const float* seg[(NT - 1) / RSEG + 1];
  seg[0] = base;
#pragma unroll
  for (int s = 1; s <= (NT - 1) / RSEG; ++s) seg[s] = base + opaque_int(16 * s * RSEG * C::PITCH);
  float f[C::NW];
#pragma unroll
  for (int ww = 0; ww < C::NW; ++ww) f[ww] = __int_as_float(uniform(__float_as_int(split_notes<D>(W, half)[ww])));
  halfx8 h[AHEAD + 1], l[AHEAD + 1];
  auto fetch = [&](auto X) {
    constexpr int x = decltype(X)::value, r = x / NQ, q = x % NQ;
    const float* const o = seg[r / RSEG] + 16 * (r % RSEG) * C::PITCH + 16 * q;
    h[x % (AHEAD + 1)] = *reinterpret_cast<const halfx8*>(o);
    l[x % (AHEAD + 1)] = *reinterpret_cast<const halfx8*>(o + D / 2);
  };
  static_for<0, AHEAD>([&](auto X) { fetch(X); });
  floatx4 t[2][CT];
  auto finish = [&](auto R) {
    constexpr int r = decltype(R)::value;
    const float u = SIGN * f[r / C::RB] * b.inv;
#pragma unroll
    for (int k = 0; k < CT; ++k)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float x = t[r & 1][k][v];
        acc[r][k][v] = ADD ? __builtin_fmaf(x, u, acc[r][k][v]) : x * u;
      }
  };
  static_for<0, NX>([&](auto X) {
    constexpr int x = decltype(X)::value, r = x / NQ, q = x % NQ, cur = x % (AHEAD + 1);
    if constexpr (x + AHEAD < NX) {
      fetch(IntC<x + AHEAD>{});
      TTC_SCHED_BARRIER();
    }
    if constexpr (q == 0)
#pragma unroll
      for (int k = 0; k < CT; ++k) t[r & 1][k] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < CT; ++k) {
      t[r & 1][k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(l[cur], b.h[q][k], t[r & 1][k], 0, 0, 0);
      t[r & 1][k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(h[cur], b.l[q][k], t[r & 1][k], 0, 0, 0);
      t[r & 1][k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(h[cur], b.h[q][k], t[r & 1][k], 0, 0, 0);
    }
    if constexpr (q == 0 && r > 0) finish(IntC<r - 1>{});
    TTC_SCHED_BARRIER();
  });
  finish(IntC<NT - 1>{});
}

}  // namespace ttc
