// One backward step of the Riccati recursion with every matrix held by columns, and the dense solve that goes with it.
//
// The accumulator layout of a 16 x 16 tile (lane 16 g + i holds M[4g + v][i], v = 0..3) is at once its B operand when the
// contraction index is visited as k = 4 g + t.  A wavefront that owns whole columns of a product therefore holds, without
// a move, the right operand of the next one: P A, then B^T (P A) and A^T (P A), then S^{-1} (B^T P A) run from register to
// register, and LDS holds left operands only, each read 16 bytes a lane for 4 RB matrix instructions.  (Owning rows
// instead, every product passes through LDS and every wavefront reads every right operand.)
//
// The products of d >= 32 run on the float16 matrix cores from split operands (ttc_split.hpp): the registers a split leaves are a
// right operand and, stored as they are, the left operand of the transpose.  Taking the diagonal's signs E out of A (P A = P E +
// P (A - E), A^T Y = E Y + (A - E)^T Y; none where the entry is below 1/2) costs one addition in the accumulator and leaves the product with what is small where the
// dynamics are near the identity; gradients of 8 steps at d = 64 are off by 0.7 times what float32 products gave (24 steps: 0.6).
//
// Measured, T = 8, float32, float32 products -> split -> split, with the inverse of a pivot block by blocks of four pivots and the
// wavefront on the serial chain at a higher priority: roll-out d = 64, 4096 problems 1.36 -> 0.99 -> 0.94 ms; backward pass d = 64, 8192
// problems 2.91 -> 2.29 -> 2.20.  Float32 products -> split: roll-out d = 32, 8192 problems 0.44 -> 0.40, d = 128, 512 problems 1.42 ->
// 0.92; ttc_lqr_solve_tv d = 64, 1024 problems 0.36 -> 0.29; at d = 32 and 1024 problems, where a step alone counts, 0.081 -> 0.090.
// What is left at d = 64 is the dense solve's serial chain, half of a step, hidden as far as three workgroups a compute unit allow.
#pragma once
#include "ttc_common.hpp"
#include "ttc_small.hpp"
#include "ttc_split.hpp"

namespace ttc {

// Workgroup barrier that orders LDS accesses only: global loads stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Wavefronts per SIMD that the registers of a kernel built on these steps are kept small enough for: with one column tile
// a wavefront at d = 64 three workgroups fit a compute unit (four spill), as do three wavefronts a SIMD at d <= 32.
#ifndef TTC_COLS_WAVES
#define TTC_COLS_WAVES(D) ((D) == 64 && Cfg<D>::RB == 1 ? 3 : (D) <= 32 ? 3 : 1)
#endif

// A d x d matrix by columns: wavefront w owns the column tiles RB w + k, tile (r, k) of it is m[r][k].
template <int D, int CT = Cfg<D>::RB>
using Cols = floatx4[Cfg<D>::NT][CT];

template <int D, int CT>
__device__ __forceinline__ void zero_cols(floatx4 (&m)[D / 16][CT]) {
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int k = 0; k < CT; ++k) m[r][k] = floatx4{0.f, 0.f, 0.f, 0.f};
}
// The sign (1 or -1) of an entry on A's diagonal, 0 for one below 1/2 (it would take more out of a small column than there is in it).
__device__ __forceinline__ float diagonal_sign(float x) { return __builtin_fabsf(x) >= 0.5f ? __builtin_copysignf(1.f, x) : 0.f; }
// m -= diag(e), e for a lane's columns
template <int D>
__device__ __forceinline__ void subtract_diagonal(Cols<D>& m, const float (&e)[Cfg<D>::RB], int w, int i, int g) {
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int k = 0; k < Cfg<D>::RB; ++k)
#pragma unroll
      for (int v = 0; v < 4; ++v) m[r][k][v] -= (r == Cfg<D>::RB * w + k && 4 * g + v == i) ? e[k] : 0.f;
}
// the largest of a non-negative value's copies in the four lane groups that hold a column (as bits: NaN on top)
__device__ __forceinline__ float column_max(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const uint32_t y = h[0] > h[1] ? h[0] : h[1];
  const auto q = __builtin_amdgcn_permlane16_swap(y, y, false, false);
  return __uint_as_float(q[0] > q[1] ? q[0] : q[1]);
}
// the largest magnitudes of a lane's columns
template <int D>
__device__ __forceinline__ void column_sizes(const Cols<D>& m, float (&x)[Cfg<D>::RB]) {
#pragma unroll
  for (int k = 0; k < Cfg<D>::RB; ++k) {
    float big = 0.f;
#pragma unroll
    for (int r = 0; r < D / 16; ++r)
#pragma unroll
      for (int v = 0; v < 4; v += 2)
        big = __builtin_fmaxf(big, __builtin_fmaxf(__builtin_fabsf(m[r][k][v]), __builtin_fabsf(m[r][k][v + 1])));
    x[k] = column_max(big);
  }
}
// the magnitudes of the diagonal entries of a lane's columns, in all four groups
template <int D>
__device__ __forceinline__ void diagonal_sizes(const Cols<D>& m, float (&x)[Cfg<D>::RB], int w, int i, int g) {
#pragma unroll
  for (int k = 0; k < Cfg<D>::RB; ++k) {
    float d = 0.f;
#pragma unroll
    for (int r = 0; r < D / 16; ++r)
#pragma unroll
      for (int v = 0; v < 4; ++v) d = (r == Cfg<D>::RB * w + k && 4 * g + v == i) ? __builtin_fabsf(m[r][k][v]) : d;
    x[k] = column_max(d);
  }
}
// the power of two above a magnitude, from 2^-80 to 2^80
__device__ __forceinline__ float unit_above(float x) {
  uint32_t u = (__float_as_uint(x) & 0x7F800000u) + (1u << 23);
  u = u < (47u << 23) ? 47u << 23 : (u > (207u << 23) ? 207u << 23 : u);
  return __uint_as_float(u);
}
// Whether the d values in LDS (as float bits, none negative) span more than a factor of 2^BITS; all wavefronts agree.
template <int D, int BITS>
__device__ __forceinline__ bool spread_above(const float* u, int g) {
  uint32_t lo = ~0u, hi = 0u;
#pragma unroll
  for (int r = 0; r < D / 16; ++r) {
    const floatx4 x = *reinterpret_cast<const floatx4*>(u + 16 * r + 4 * g);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const uint32_t b = __float_as_uint(x[v]);
      lo = b < lo ? b : lo;
      hi = b > hi ? b : hi;
    }
  }
  hi = __float_as_uint(column_max(__uint_as_float(hi)));
  lo = ~__float_as_uint(column_max(__uint_as_float(~lo)));
  return uniform((int)(hi - lo)) > (BITS << 23);
}
// m <- diag(u) m or diag(1 / u) m, u a vector of powers of two in LDS (INVERSE) or of any numbers
template <int D, bool INVERSE = false>
__device__ __forceinline__ void scale_rows(Cols<D>& m, const float* u, int g) {
#pragma unroll
  for (int r = 0; r < D / 16; ++r) {
    floatx4 x = *reinterpret_cast<const floatx4*>(u + 16 * r + 4 * g);
    if (INVERSE)
#pragma unroll
      for (int v = 0; v < 4; ++v) x[v] = power_inverse(x[v]);
#pragma unroll
    for (int k = 0; k < Cfg<D>::RB; ++k) m[r][k] = m[r][k] * x;
  }
}
// m <- m diag(x)
template <int D>
__device__ __forceinline__ void scale_columns(Cols<D>& m, const float (&x)[Cfg<D>::RB]) {
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int k = 0; k < Cfg<D>::RB; ++k) m[r][k] = m[r][k] * x[k];
}
// The power of two whose square is above x >= 0 and at most 4 x (2^80 at most, also for what is not finite).
__device__ __forceinline__ float unit_of_square(float x) {
  const uint32_t e = __float_as_uint(x) >> 23;  // 127 + e
  const uint32_t u = (((e + 127u) >> 1) + 1u) << 23;
  return __uint_as_float(u < (207u << 23) ? u : 207u << 23);
}
// From a row-major matrix in memory, as read: a row of 16 lanes reads 16 consecutive elements; of the transpose a lane's four entries
// are consecutive.
template <int D, typename TIn>
struct ReadCols {
  decltype(read1((const TIn*)nullptr, 0)) x[D / 16][Cfg<D>::RB][4];
  __device__ __forceinline__ void read(const TIn* M, int w, int i, int g) {
    const unsigned o = (unsigned)(4 * g * D + 16 * Cfg<D>::RB * w + i);
#pragma unroll
    for (int r = 0; r < D / 16; ++r)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int k = 0; k < Cfg<D>::RB; ++k) x[r][k][v] = read1(M, o + (unsigned)((16 * r + v) * D + 16 * k));
  }
  __device__ __forceinline__ void to(Cols<D>& m) const {
#pragma unroll
    for (int r = 0; r < D / 16; ++r)
#pragma unroll
      for (int k = 0; k < Cfg<D>::RB; ++k)
#pragma unroll
        for (int v = 0; v < 4; ++v) m[r][k][v] = widen(x[r][k][v]);
  }
};
template <int D, typename TIn>
struct ReadColsT {
  decltype(read4((const TIn*)nullptr, 0)) x[D / 16][Cfg<D>::RB];
  __device__ __forceinline__ void read(const TIn* M, int w, int i, int g) {
    const unsigned o = (unsigned)((16 * Cfg<D>::RB * w + i) * D + 4 * g);
#pragma unroll
    for (int r = 0; r < D / 16; ++r)
#pragma unroll
      for (int k = 0; k < Cfg<D>::RB; ++k) x[r][k] = read4(M, o + (unsigned)(16 * k * D + 16 * r));
  }
};
template <int D, typename TIn>
__device__ __forceinline__ void load_cols(const TIn* M, Cols<D>& m, int w, int i, int g) {
  ReadCols<D, TIn> t;
  t.read(M, w, i, g);
  TTC_SCHED_BARRIER();
  t.to(m);
}
template <int D, typename TIn>
__device__ __forceinline__ void load_cols_T(const TIn* M, Cols<D>& m, int w, int i, int g) {
  ReadColsT<D, TIn> t;
  t.read(M, w, i, g);
  TTC_SCHED_BARRIER();
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int k = 0; k < Cfg<D>::RB; ++k) m[r][k] = widen(t.x[r][k]);
}
template <int D>
__device__ __forceinline__ void eye_cols(Cols<D>& m, int w, int i, int g) {
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int k = 0; k < Cfg<D>::RB; ++k)
#pragma unroll
      for (int v = 0; v < 4; ++v) m[r][k][v] = (r == Cfg<D>::RB * w + k && 4 * g + v == i) ? 1.f : 0.f;
}
// m += the symmetric part of such a matrix (the transposed entries of a lane are four consecutive elements)
template <int D, typename TIn>
__device__ __forceinline__ void add_sym_cols(const TIn* M, Cols<D>& m, int w, int i, int g) {
  ReadCols<D, TIn> t;
  ReadColsT<D, TIn> tt;
  t.read(M, w, i, g);
  tt.read(M, w, i, g);
  TTC_SCHED_BARRIER();
  Cols<D> c;
  t.to(c);
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int k = 0; k < Cfg<D>::RB; ++k) m[r][k] += 0.5f * (c[r][k] + widen(tt.x[r][k]));
}
// A matrix by columns to memory and back as it stands in the registers, 16 bytes a lane: of a matrix that every step reads
// (time-invariant parameters), its symmetric part takes a fifth of the reads this way.
template <int D>
__device__ __forceinline__ void keep_cols(float* M, const Cols<D>& m, int tid) {
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int k = 0; k < Cfg<D>::RB; ++k)
      reinterpret_cast<floatx4*>(M)[(r * Cfg<D>::RB + k) * Cfg<D>::NTHR + tid] = m[r][k];
}
template <int D>
__device__ __forceinline__ void add_kept_cols(const float* M, Cols<D>& m, int tid) {
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int k = 0; k < Cfg<D>::RB; ++k)
      m[r][k] += reinterpret_cast<const floatx4*>(M)[(r * Cfg<D>::RB + k) * Cfg<D>::NTHR + tid];
}
// the transpose (times SIGN) to LDS, row-major: a lane's four values are 16 bytes of one row
template <int D, int SIGN = 1>
__device__ __forceinline__ void store_cols_T(float* L, const Cols<D>& m, int w, int i, int g) {
  float* const o = L + (16 * Cfg<D>::RB * w + i) * Cfg<D>::PITCH + 4 * g;
#pragma unroll
  for (int k = 0; k < Cfg<D>::RB; ++k)
#pragma unroll
    for (int r = 0; r < D / 16; ++r)
      *reinterpret_cast<floatx4*>(o + 16 * k * Cfg<D>::PITCH + 16 * r) = SIGN > 0 ? m[r][k] : -m[r][k];
}
// the matrix itself to LDS (row pitch PITCH) or to memory (row pitch D), row-major
template <int D, int SIGN = 1>
__device__ __forceinline__ void store_cols(float* L, int pitch, const Cols<D>& m, int w, int i, int g) {
  float* const o = L + 4 * g * pitch + 16 * Cfg<D>::RB * w + i;
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int k = 0; k < Cfg<D>::RB; ++k) o[(16 * r + v) * pitch + 16 * k] = SIGN > 0 ? m[r][k][v] : -m[r][k][v];
}

// from LDS (row pitch PITCH), the matrix itself and its transpose
template <int D>
__device__ __forceinline__ void read_cols(const float* L, Cols<D>& m, int w, int i, int g) {
  const float* const o = L + 4 * g * Cfg<D>::PITCH + 16 * Cfg<D>::RB * w + i;
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int k = 0; k < Cfg<D>::RB; ++k) m[r][k][v] = o[(16 * r + v) * Cfg<D>::PITCH + 16 * k];
}
template <int D>
__device__ __forceinline__ void read_cols_T(const float* L, Cols<D>& m, int w, int i, int g) {
  const float* const o = L + (16 * Cfg<D>::RB * w + i) * Cfg<D>::PITCH + 4 * g;
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int k = 0; k < Cfg<D>::RB; ++k) m[r][k] = *reinterpret_cast<const floatx4*>(o + 16 * k * Cfg<D>::PITCH + 16 * r);
}

// acc += L R: L row-major in LDS, R by columns.  The left operand of the next four k-steps is read while the current ones
// run; scheduling barriers keep the compiler from hoisting more reads than that.
template <int D, int CT>
__device__ __forceinline__ void gemm_cols(floatx4 (&acc)[D / 16][CT], const float* L, const floatx4 (&b)[D / 16][CT], int i,
                                          int g) {
  using C = Cfg<D>;
  constexpr int NT = C::NT;
  // rows of one base register (an LDS instruction carries a 16-bit byte offset)
  constexpr int RSEG = 65000 / (16 * C::PITCH * 4) > 0 ? 65000 / (16 * C::PITCH * 4) : 1;
  const float* const base = L + i * C::PITCH + 4 * g;
  const float* seg[(NT - 1) / RSEG + 1];
  seg[0] = base;
#pragma unroll
  for (int s = 1; s <= (NT - 1) / RSEG; ++s) seg[s] = base + opaque_int(16 * s * RSEG * C::PITCH);
  floatx4 a[2];
  a[0] = *reinterpret_cast<const floatx4*>(base);
  static_for<0, NT * NT>([&](auto X) {
    constexpr int x = decltype(X)::value, r = x / NT, q = x % NT, cur = x & 1;
    if constexpr (x + 1 < NT * NT) {
      constexpr int r1 = (x + 1) / NT, q1 = (x + 1) % NT;
      a[cur ^ 1] = *reinterpret_cast<const floatx4*>(seg[r1 / RSEG] + 16 * (r1 % RSEG) * C::PITCH + 16 * q1);
      TTC_SCHED_BARRIER();
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int k = 0; k < CT; ++k)
        acc[r][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[cur][t], b[q][k][t], acc[r][k], 0, 0, 0);
    TTC_SCHED_BARRIER();
  });
}

// f(p) for p = 0, CT, .. below NT: a loop from eight blocks on, their code one after the other below.
template <int NT, int CT, typename F>
__device__ __forceinline__ void for_each_block(F&& f) {
  if constexpr (NT >= 8) {
#pragma unroll 1
    for (int p = 0; p < NT; p += CT) f(p);
  } else {
    static_for<0, NT / CT>([&](auto X) { f(decltype(X)::value * CT); });
  }
}

// Dense solve f <- s^{-1} f, both by columns (f: FT column tiles a wavefront, also none), for a symmetric positive definite s,
// or any whose elimination in order meets pivots above piv_min only: block Gauss-Jordan with 16 x 16 pivot blocks and no pivot
// search.  Per block p, the wavefront that owns its columns
// inverts s[p][p] in registers and publishes that inverse and the rest of the column, negated, as left operands (Wp: the
// right half of the pair); every wavefront then does its own columns, U = s[p][p]^{-1} s[p][c], s[r][c] -= s[r][p] U,
// the next block's first, so that its inverse is formed and published under the others' updates: one workgroup barrier
// per block, no right operand through LDS, and a serial chain of some 1500 cycles per 16 columns (the pivoted panels of
// lds_solve: about 5000).  The wavefront on that chain has priority over the others of its SIMD, of this problem and of others (d = 64:
// squaring T = 8, 16384 problems 2.40 -> 2.31 ms, roll-out T = 8, 4096 problems 0.986 -> 0.959; at d = 128 no difference).
// With d <= 32 the explicit inverse alone loses up to a factor of three where control is cheap (the block is most of the
// matrix); there one step of refinement, U += s[p][p]^{-1} (s[p][c] - s[p][p] U), restores a factor-and-solve's accuracy
// (REFINE).  From d = 64 on the recursion does not show it (measured against float64, cost ratios 1 to 1e4), but a single
// solve does: the backward pass asks for it in its first step's, where it costs nothing beside the steps.
// Returns, uniformly, whether a pivot was not above piv_min and finite.  Wp must be free to every wavefront on entry; its last
// reads may still be under way in other wavefronts on return.
// Row tiles turn by one place a block, so that the pivot block is tile 0 of its column and block p + r tile r, in registers (a
// matrix instruction adds tile r into the place of tile r - 1) as in LDS: at d = 128 the loop over the blocks is one.  Unrolled there,
// a solve is five thousand instructions, and a kernel of several fetches them from memory each time (roll-out d = 128, T = 8, 1024
// problems 2.08 -> 1.74 ms, backward pass 2.75 -> 2.28, squaring T = 16, 8192 problems 11.6 -> 11.0); at d = 64 the loop is the
// slower of the two (squaring T = 8, 16384 problems 2.55 -> 2.63 ms).
template <int D, int FT, bool REFINE = (D <= 32)>
__device__ __forceinline__ int solve_cols(float* Wp, Cols<D>& s, floatx4 (&f)[D / 16][FT > 0 ? FT : 1], int w, int lane,
                                          float piv_min = 0.f) {
  using C = Cfg<D>;
  constexpr int NT = C::NT, CT = C::RB;
  constexpr bool LOCAL = C::NW == 1;  // one wavefront: the refinement's operand stays in it
  // The pivot block's inverse by blocks of four pivots, or by columns.  At d = 128 a wavefront holds eight tiles beside it, and -M^T and the panel
  // of four make registers spill around it that the columns leave alone (solve_tv_kernel 104 / 83, T = 8, 1024 problems 2.05 / 1.90 ms; the
  // recursion behind squaring, T = 16, 512 problems 2.01 / 1.87; roll-out, 512 problems of 6 steps, 0.694 / 0.706).
  constexpr bool BLOCKS = D < 128;
  const int i = lane & 15, g = lane >> 4;
  w = uniform(w);
  int bad = 0;
  floatx4 d_neg;  // REFINE: minus the pivot block, as a left operand
  auto publish = [&](auto K, int buf) {  // by the wavefront that owns the column tile
    constexpr int k = decltype(K)::value;
    float* const o = Wp + 4 * g * C::PITCH + 16 * buf + i;
    if constexpr (REFINE && LOCAL) {  // through the tile the inverse goes to below (a wavefront's LDS operations run in order)
#pragma unroll
      for (int v = 0; v < 4; ++v) o[v * C::PITCH] = -s[0][k][v];
      wave_lds_sync();
      d_neg = *reinterpret_cast<const floatx4*>(Wp + i * C::PITCH + 16 * buf + 4 * g);
      wave_lds_sync();
    } else if constexpr (REFINE) {  // to the columns behind both buffers' inverses
#pragma unroll
      for (int v = 0; v < 4; ++v) o[32 + v * C::PITCH] = -s[0][k][v];
    }
    floatx4 inv = s[0][k];
    if constexpr (BLOCKS) bad |= invert_spread16(inv, Wp + 16 * buf, C::PITCH, lane, piv_min);
    else bad |= invert_columns16(inv, lane, piv_min);
#pragma unroll
    for (int r = 0; r < NT; ++r) {
      const floatx4 x = r == 0 ? inv : -s[r][k];
#pragma unroll
      for (int v = 0; v < 4; ++v) o[(16 * r + v) * C::PITCH] = x[v];
    }
  };
  auto column = [&](const floatx4 (&x)[NT], auto& m, auto K, int p) {
    constexpr int k = decltype(K)::value;
    floatx4 u = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) u = __builtin_amdgcn_mfma_f32_16x16x4f32(x[0][t], m[0][k][t], u, 0, 0, 0);
    if constexpr (REFINE) {
      floatx4 res = m[0][k];
#pragma unroll
      for (int t = 0; t < 4; ++t) res = __builtin_amdgcn_mfma_f32_16x16x4f32(d_neg[t], u[t], res, 0, 0, 0);
#pragma unroll
      for (int t = 0; t < 4; ++t) u = __builtin_amdgcn_mfma_f32_16x16x4f32(x[0][t], res[t], u, 0, 0, 0);
    }
    if constexpr (FT > 0) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 1; r < NT; ++r)
          m[r - 1][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[r][t], u[t], t == 0 ? m[r][k] : m[r - 1][k], 0, 0, 0);
    } else {  // without right-hand sides the rows of blocks already taken are not needed
#pragma unroll
      for (int r = 1; r < NT; ++r)
        if (r < NT - p)
#pragma unroll
          for (int t = 0; t < 4; ++t)
            m[r - 1][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[r][t], u[t], t == 0 ? m[r][k] : m[r - 1][k], 0, 0, 0);
    }
    m[NT - 1][k] = u;
  };
  if (w == 0) publish(IntC<0>{}, 0);
  for_each_block<NT, CT>([&](int p0) {
    static_for<0, CT>([&](auto KK) {
      constexpr int kk = decltype(KK)::value, kn = (kk + 1) % CT;  // the pivot block's tile in its wavefront, and the next one's
      const int p = p0 + kk, buf = p & 1;
      lds_barrier();  // block p is published; block p - 1 (the other buffer) was read before
      floatx4 x[NT];
#pragma unroll
      for (int r = 0; r < NT; ++r) x[r] = *reinterpret_cast<const floatx4*>(Wp + (16 * r + i) * C::PITCH + 16 * buf + 4 * g);
      if constexpr (REFINE && !LOCAL) d_neg = *reinterpret_cast<const floatx4*>(Wp + i * C::PITCH + 32 + 16 * buf + 4 * g);
      const bool next_here = p + 1 < NT && w == (p + 1) / CT;
      auto rest = [&] {
        static_for<0, CT>([&](auto K) {
          constexpr int k = decltype(K)::value;
          if (CT * w + k > p && !(k == kn && next_here)) column(x, s, K, p);
        });
        if constexpr (FT > 0) static_for<0, FT>([&](auto K) { column(x, f, K, p); });
      };
      if constexpr (REFINE && LOCAL) {  // the others still need this block's operands
        if (next_here) column(x, s, IntC<kn>{}, p);
        rest();
        if (next_here) publish(IntC<kn>{}, buf ^ 1);
      } else {
        if (next_here) {
          __builtin_amdgcn_s_setprio(3);  // the others' updates are not waited for by anyone
          column(x, s, IntC<kn>{}, p);
          publish(IntC<kn>{}, buf ^ 1);
          __builtin_amdgcn_s_setprio(0);
        }
        rest();
      }
    });
  });
  // the wavefronts' flags meet in the skew columns of the pair, which nothing else uses
  const int any = __any(bad) ? 1 : 0;
  if constexpr (C::NW == 1) {
    lds_barrier();
    return any;
  } else {
    int* const flags = reinterpret_cast<int*>(Wp + D);
    if (lane == 0) flags[w * C::PITCH] = any;
    lds_barrier();
    int all = 0;
#pragma unroll
    for (int ww = 0; ww < C::NW; ++ww) all |= flags[ww * C::PITCH];
    return uniform(all);
  }
}

// s <- s^{-1} by the same elimination in place: the column of a pivot block becomes that of the inverse as soon as it has been
// used, so that no right-hand sides are carried (two thirds of the work of solving for the identity, and its registers).
// With d <= 32, where a block's explicit inverse is not accurate enough, the identity is solved for.
template <int D>
__device__ __forceinline__ int invert_cols(float* Wp, Cols<D>& s, int w, int lane, float piv_min) {
  using C = Cfg<D>;
  constexpr int NT = C::NT, CT = C::RB;
  const int i = lane & 15, g = lane >> 4;
  w = uniform(w);
  if constexpr (D <= 32) {
    Cols<D> f;
    eye_cols<D>(f, w, i, g);
    const int flag = solve_cols<D, CT>(Wp, s, f, w, lane, piv_min);
#pragma unroll
    for (int r = 0; r < NT; ++r)
#pragma unroll
      for (int k = 0; k < CT; ++k) s[r][k] = f[r][k];
    return flag;
  }
  int bad = 0;
  auto publish = [&](auto K, int buf) {  // by the wavefront that owns the column tile
    constexpr int k = decltype(K)::value;
    float* const o = Wp + 4 * g * C::PITCH + 16 * buf + i;
#pragma unroll
    for (int r = 1; r < NT; ++r)
#pragma unroll
      for (int v = 0; v < 4; ++v) o[(16 * r + v) * C::PITCH] = -s[r][k][v];
    bad |= invert_spread16(s[0][k], Wp + 16 * buf, C::PITCH, lane, piv_min);
#pragma unroll
    for (int v = 0; v < 4; ++v) o[v * C::PITCH] = s[0][k][v];
  };
  // own: the pivot block's column, whose inverse stands in s[0][k]; the rest becomes -s[r][p] times that
  auto column = [&](const floatx4 (&x)[NT], auto K, bool own) {
    constexpr int k = decltype(K)::value;
    floatx4 u = s[0][k];
    if (!own) {
      u = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 4; ++t) u = __builtin_amdgcn_mfma_f32_16x16x4f32(x[0][t], s[0][k][t], u, 0, 0, 0);
    } else {
#pragma unroll
      for (int r = 1; r < NT; ++r) s[r][k] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 1; r < NT; ++r)
        s[r - 1][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[r][t], u[t], t == 0 ? s[r][k] : s[r - 1][k], 0, 0, 0);
    s[NT - 1][k] = u;
  };
  if (w == 0) publish(IntC<0>{}, 0);
  for_each_block<NT, CT>([&](int p0) {
    static_for<0, CT>([&](auto KK) {
      constexpr int kk = decltype(KK)::value, kn = (kk + 1) % CT;
      const int p = p0 + kk, buf = p & 1;
      lds_barrier();  // block p is published; block p - 1 (the other buffer) was read before
      floatx4 x[NT];
#pragma unroll
      for (int r = 0; r < NT; ++r) x[r] = *reinterpret_cast<const floatx4*>(Wp + (16 * r + i) * C::PITCH + 16 * buf + 4 * g);
      const bool next_here = p + 1 < NT && w == (p + 1) / CT;
      if (next_here) {
        __builtin_amdgcn_s_setprio(3);
        column(x, IntC<kn>{}, false);
        publish(IntC<kn>{}, buf ^ 1);
        __builtin_amdgcn_s_setprio(0);
      }
      static_for<0, CT>([&](auto K) {
        constexpr int k = decltype(K)::value;
        if (!(k == kn && next_here)) column(x, K, CT * w + k == p);
      });
    });
  });
  const int any = __any(bad) ? 1 : 0;
  int* const flags = reinterpret_cast<int*>(Wp + D);
  if (lane == 0) flags[w * C::PITCH] = any;
  lds_barrier();
  int all = 0;
#pragma unroll
  for (int ww = 0; ww < C::NW; ++ww) all |= flags[ww * C::PITCH];
  return uniform(all);
}

// Units of the states for the products of a step, as powers of two: the unit D_j of state j is just above max_i |P_ij| / sqrt(P_ii),
// which is sqrt(P_jj) where P is semidefinite (and no less than half of sqrt(max_i |P_ij|) where P_jj is 0).  Written x' = D x, all
// entries of P are below 2 whatever the units of the problem, and a product over the states adds terms of like weight.
template <int D>
__device__ __forceinline__ void publish_state_units(Pair<D>& W, const Cols<D>& P, int w, int i, int g) {
  using C = Cfg<D>;
  float* const aux = control_units<D>(W);
  float x[C::RB], c[C::RB];
  diagonal_sizes<D>(P, x, w, i, g);
  column_sizes<D>(P, c);
#pragma unroll
  for (int k = 0; k < C::RB; ++k) {
    x[k] = unit_of_square(x[k] == 0.f ? c[k] : x[k]);
    aux[16 * (C::RB * w + k) + i] = power_inverse(x[k]);
  }
  lds_barrier();
#pragma unroll
  for (int k = 0; k < C::RB; ++k) {
    float big = __uint_as_float(__float_as_uint(0.5f * x[k]) - 1u);  // (just below, as unit_above goes to the next power)
#pragma unroll
    for (int r = 0; r < C::NT; ++r) {
      const floatx4 y = *reinterpret_cast<const floatx4*>(aux + 16 * r + 4 * g);
#pragma unroll
      for (int v = 0; v < 4; ++v) big = __builtin_fmaxf(big, __builtin_fabsf(P[r][k][v]) * y[v]);
    }
    state_units<D>(W)[16 * (C::RB * w + k) + i] = unit_above(column_max(big));
  }
  lds_barrier();
}
// The spread of positive values as a pair of 16-bit numbers of which maxima are taken: the exponent, and 255 less it.
typedef unsigned short ushortx2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t spread_of(float x) {
  const uint32_t e = __float_as_uint(x) >> 23;
  return e | (255u - e) << 16;
}
__device__ __forceinline__ uint32_t spread_join(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ushortx2, a), __builtin_bit_cast(ushortx2, b)));
}
__device__ __forceinline__ uint32_t spread_join16(uint32_t x) {  // over the sixteen lanes of a group
  x = spread_join(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
  x = spread_join(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
  x = spread_join(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, false));  // row_half_mirror
  return spread_join(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xF, 0xF, false));  // row_mirror
}
__device__ __forceinline__ int spread_bits(uint32_t x) { return (int)(x & 0xFFFFu) + (int)(x >> 16) - 255; }  // (-255: all zero)
// Whether the operands of a step need units of their own: the diagonal of P spans more than a factor of 2^14, or the columns of B or
// of A (e: the signs taken out of t) more than 2^7; up to there the digits that split operands have beyond float32 do.  One barrier,
// which all wavefronts reach with P read; it and the judgement cost 2 to 4 % of a step (ttc_lqr_solve_tv, d = 64, T = 8, 8192 problems 1.86
// -> 1.92 ms).
template <int D>
__device__ __forceinline__ bool step_needs_units(Pair<D>& W, const Cols<D>& P, const Cols<D>& B, const Cols<D>& t,
                                                 const float (&e)[Cfg<D>::RB], int w, int i, int g) {
  using C = Cfg<D>;
  uint32_t* const judge = reinterpret_cast<uint32_t*>(column_units<D>(W));
  float x[3][C::RB];
  diagonal_sizes<D>(P, x[0], w, i, g);
  column_sizes<D>(B, x[1]);
  column_sizes<D>(t, x[2]);
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < C::RB; ++k) {
      if (q == 2) x[q][k] = __builtin_fmaxf(x[q][k], __builtin_fabsf(e[k]));
      // (a column of zeros has no size; a state without a cost has rows of B and A that must not set the scale)
      s = spread_join(s, q > 0 && x[q][k] == 0.f ? 0u : spread_of(x[q][k]));
    }
    judge[3 * w + q] = spread_join16(s);
  }
  lds_barrier();
  uint32_t s[3] = {0, 0, 0};
#pragma unroll
  for (int ww = 0; ww < C::NW; ++ww)
#pragma unroll
    for (int q = 0; q < 3; ++q) s[q] = spread_join(s[q], judge[3 * ww + q]);
  const int p = uniform(spread_bits(s[0])), b = uniform(spread_bits(s[1])), a = uniform(spread_bits(s[2]));
  return p > 14 || b > 7 || a > 7;
}

// P, B, R (in s) and A - E (in t) of a step in units of its own, with D E C^{-1} in the place of E.  V and C go behind the pair.
template <int D>
__device__ __forceinline__ void step_in_units(Pair<D>& W, Cols<D>& P, Cols<D>& B, Cols<D>& s, Cols<D>& t, float (&e)[Cfg<D>::RB],
                                              int w, int i, int g) {
  using C = Cfg<D>;
  lds_barrier();
  publish_state_units<D>(W, P, w, i, g);
  const float* const units = state_units<D>(W);
  float x[C::RB], y[C::RB], u[C::RB];
#pragma unroll
  for (int k = 0; k < C::RB; ++k) {
    u[k] = units[16 * (C::RB * w + k) + i];
    x[k] = power_inverse(u[k]);
  }
  scale_rows<D, true>(P, units, g);
  scale_columns<D>(P, x);
  // V: the largest entry of a column of D B is in [1, 2), and that of R at most 2^80
  scale_rows<D>(B, units, g);
  column_sizes<D>(B, x);
  diagonal_sizes<D>(s, y, w, i, g);
#pragma unroll
  for (int k = 0; k < C::RB; ++k) {
    const float v = __builtin_fmaxf(0.5f * unit_above(x[k]), __builtin_ldexpf(unit_of_square(y[k]), -40));
    control_units<D>(W)[16 * (C::RB * w + k) + i] = v;
    x[k] = power_inverse(v);
  }
  // C: a column of D A is of the size of the larger of D E and D (A - E)
  scale_rows<D>(t, units, g);
  column_sizes<D>(t, y);
#pragma unroll
  for (int k = 0; k < C::RB; ++k) {
    const float big = __builtin_fmaxf(y[k], __builtin_fabsf(e[k]) * u[k]);
    const float c = big == 0.f ? 1.f : unit_above(big);
    column_units<D>(W)[16 * (C::RB * w + k) + i] = c;
    y[k] = power_inverse(c);
    e[k] *= u[k] * y[k];
  }
  scale_columns<D>(t, y);
  lds_barrier();
  scale_columns<D>(B, x);
  scale_columns<D>(s, x);
  scale_rows<D, true>(s, control_units<D>(W), g);
}

// The operands of a step at d >= 32, by columns: P (symmetric, from the right half of the pair), B, R (through add_R), E and A - E.
template <int D, typename TIn, typename AddR>
__device__ __forceinline__ void step_operands(Pair<D>& W, const TIn* As, const TIn* Bs, AddR&& add_R, Cols<D>& P, Cols<D>& B,
                                              Cols<D>& s, Cols<D>& t, float (&e)[Cfg<D>::RB], int w, int i, int g) {
  using C = Cfg<D>;
  {
    ReadCols<D, TIn> b, a;
    decltype(read1(As, 0)) d[C::RB];
    b.read(Bs, w, i, g);
    a.read(As, w, i, g);
#pragma unroll
    for (int k = 0; k < C::RB; ++k) d[k] = read1(As, (long)(16 * (C::RB * w + k) + i) * (D + 1));
    zero_cols<D>(s);
    TTC_SCHED_BARRIER();
    add_R(s, w, i, g);
    TTC_SCHED_BARRIER();  // the step's reads are all under way
    b.to(B);
    a.to(t);
#pragma unroll
    for (int k = 0; k < C::RB; ++k) e[k] = diagonal_sign(widen(d[k]));
  }
  // P is symmetric: a lane's four entries of a column are four consecutive ones of its row
#pragma unroll
  for (int r = 0; r < C::NT; ++r)
#pragma unroll
    for (int k = 0; k < C::RB; ++k)
      P[r][k] = *reinterpret_cast<const floatx4*>(W + D + (16 * (C::RB * w + k) + i) * C::PITCH + 16 * r + 4 * g);
  subtract_diagonal<D>(t, e, w, i, g);
}
// Its six products and the solve, from these operands (P is replaced, every wavefront has read it).
template <int D>
__device__ __forceinline__ int step_products(Pair<D>& W, Cols<D>& pn, const Cols<D>& bc, Cols<D>& s, const Cols<D>& t,
                                             const float (&e)[Cfg<D>::RB], Cols<D>& wk, int w, int lane, int i, int g) {
  using C = Cfg<D>;
  using Split = SplitCols<D, C::RB>;
  constexpr int L = 0, R = 1;  // the halves
  float* const signs = diagonal_signs<D>(W);
  {
    Split a;
    {
      Split b;
      {
        Split p;
        split_cols<D, C::RB>(pn, p);
        store_split_T<D>(W, R, p, w, i, g);  // P
        split_cols<D, C::RB>(bc, b);
        store_split_T<D>(W, L, b, w, i, g);  // B^T
      }
      if (g == 0)
#pragma unroll
        for (int k = 0; k < C::RB; ++k) signs[16 * (C::RB * w + k) + i] = e[k];
      lds_barrier();
      Cols<D> pb;
      gemm_split<D, C::RB>(pb, W, R, b, i, g);  // P B
      split_cols<D, C::RB>(pb, b);
      gemm_split<D, C::RB, true>(s, W, L, b, i, g);  // S = R + B^T P B
      split_cols<D, C::RB>(t, a);
    }
    Split pa;
    scale_columns<D>(pn, e);
    gemm_split<D, C::RB, true>(pn, W, R, a, i, g);  // P A = P E + P (A - E)
    split_cols<D, C::RB>(pn, pa);
    gemm_split<D, C::RB>(wk, W, L, pa, i, g);  // F = B^T P A
    Split f;
    split_cols<D, C::RB>(wk, f);
    lds_barrier();                           // P and B^T are no longer read
    store_split_T<D>(W, R, a, w, i, g);  // (A - E)^T
    store_split_T<D>(W, L, f, w, i, g);  // F^T
    lds_barrier();
    scale_rows<D>(pn, signs, g);
    gemm_split<D, C::RB, true>(pn, W, R, pa, i, g);  // A^T P A = E P A + (A - E)^T P A
  }
  lds_barrier();
  const int flag = solve_cols<D, C::RB>(W + D, s, wk, w, lane);  // W = S^{-1} F
  Split x;
  split_cols<D, C::RB>(wk, x);
  gemm_split<D, C::RB, true, -1>(pn, W, L, x, i, g);  // - F^T W
  return flag;
}
// The same in units of the step's own, powers of two, so that results do not depend on those of the problem: x' = D x before the step's
// state, u' = V u, x' = C x behind it, and with them D^{-1} P D^{-1}, D B V^{-1}, D A C^{-1}, V^{-1} R V^{-1}.  Split operands keep 40
// binary digits below the largest entry of a wavefront's columns, float32 ones every digit of every entry: with one state in units of 2^17,
// d = 64, T = 8, u_0 was off by 3e-3 without; now by what it is in units of one, bit for bit.
// A function of its own, for the few steps that need it: inlined beside the other it costs both their registers (d = 64, T = 8, 8192
// problems 1.92 -> 2.01 ms with the scalings behind branches, 2.5 with two copies of the products).
typedef __attribute__((address_space(3))) float lds_float;
template <int D, typename TIn>
__device__ __attribute__((noinline)) int riccati_step_in_units(lds_float* pair, const TIn* As, const TIn* Bs, const TIn* Rs,
                                                               Cols<D>* wk_out, Cols<D>* pn_out, int tid) {
  using C = Cfg<D>;
  Pair<D>& W = *reinterpret_cast<Pair<D>*>((float*)pair);
  const int lane = tid & 63, w = uniform(tid >> 6), i = lane & 15, g = lane >> 4;
  Cols<D> wk, pn, bc, s, t;
  float e[C::RB];
  step_operands<D, TIn>(
      W, As, Bs, [&](Cols<D>& m, int w, int i, int g) { add_sym_cols<D, TIn>(Rs, m, w, i, g); }, pn, bc, s, t, e, w, i, g);
  step_in_units<D>(W, pn, bc, s, t, e, w, i, g);
  const int flag = step_products<D>(W, pn, bc, s, t, e, wk, w, lane, i, g);
  const float* const c = column_units<D>(W);
  float ck[C::RB];
#pragma unroll
  for (int k = 0; k < C::RB; ++k) ck[k] = c[16 * (C::RB * w + k) + i];
  scale_rows<D>(pn, c, g);
  scale_columns<D>(pn, ck);
  scale_rows<D, true>(wk, control_units<D>(W), g);
  scale_columns<D>(wk, ck);
#pragma unroll
  for (int r = 0; r < C::NT; ++r)
#pragma unroll
    for (int k = 0; k < C::RB; ++k) {
      (*wk_out)[r][k] = wk[r][k];
      (*pn_out)[r][k] = pn[r][k];
    }
  return flag;
}

// One backward step of Prop. 3.1 with the matrices of one step.  On entry the right half of the pair holds P_{s+1}
// (symmetric, visible) and the left half is free; on exit, by columns, wk = S^{-1} B^T P A = -K_s, S = R + B^T P B, and
// pn = A^T P A - (B^T P A)^T wk, which is P_s up to the stage cost.  Six products and one unpivoted solve (S is positive
// definite).  Returns the solve's breakdown flag.  Other wavefronts may still be reading the left half on return.
// add_R(s, w, i, g) adds the symmetric part of R, the matrix at Rs, to s.
template <int D, typename TIn, typename AddR>
__device__ __forceinline__ int riccati_step_with(Pair<D>& W, const TIn* As, const TIn* Bs, const TIn* Rs, AddR&& add_R, Cols<D>& wk,
                                                 Cols<D>& pn, int tid) {
  using C = Cfg<D>;
  tid += opaque_zero();
  const int lane = tid & 63, w = uniform(tid >> 6), i = lane & 15, g = lane >> 4;
  if constexpr (D == 16) {  // one tile: half of a float16 instruction's depth would be empty
    float* const WL = W;
    float* const WR = W + D;
    Cols<D> s, a, b, pb, pa;
    load_cols<D, TIn>(Bs, b, w, i, g);
    store_cols_T<D>(WL, b, w, i, g);  // B^T
    load_cols<D, TIn>(As, a, w, i, g);
    zero_cols<D>(s);
    add_R(s, w, i, g);
    lds_barrier();
    zero_cols<D>(pb);
    gemm_cols<D>(pb, WR, b, i, g);  // P B
    gemm_cols<D>(s, WL, pb, i, g);  // S = R + B^T P B
    zero_cols<D>(pa);
    gemm_cols<D>(pa, WR, a, i, g);  // P A
    zero_cols<D>(wk);
    gemm_cols<D>(wk, WL, pa, i, g);  // F = B^T P A
    lds_barrier();                 // P and B^T are no longer read
    store_cols_T<D>(WR, a, w, i, g);       // A^T
    store_cols_T<D, -1>(WL, wk, w, i, g);  // -F^T
    lds_barrier();
    zero_cols<D>(pn);
    gemm_cols<D>(pn, WR, pa, i, g);  // A^T P A
    lds_barrier();
    const int flag = solve_cols<D, C::RB>(WR, s, wk, w, lane);  // W = S^{-1} F
    gemm_cols<D>(pn, WL, wk, i, g);                                 // - F^T W
    return flag;
  } else {
    Cols<D> bc, s, t;
    float e[C::RB];
    step_operands<D, TIn>(W, As, Bs, add_R, pn, bc, s, t, e, w, i, g);
    if (__builtin_expect(step_needs_units<D>(W, pn, bc, t, e, w, i, g), 0)) {
      Cols<D> a, b;
      const int flag = riccati_step_in_units<D, TIn>((lds_float*)(float*)W, As, Bs, Rs, &a, &b, tid);
#pragma unroll
      for (int r = 0; r < C::NT; ++r)
#pragma unroll
        for (int k = 0; k < C::RB; ++k) {
          wk[r][k] = a[r][k];
          pn[r][k] = b[r][k];
        }
      return flag;
    }
    return step_products<D>(W, pn, bc, s, t, e, wk, w, lane, i, g);
  }
}

template <int D, typename TIn>
__device__ __forceinline__ int riccati_step(Pair<D>& W, const TIn* As, const TIn* Bs, const TIn* Rs, Cols<D>& wk, Cols<D>& pn,
                                            int tid) {
  return riccati_step_with<D, TIn>(
      W, As, Bs, Rs, [&](Cols<D>& s, int w, int i, int g) { add_sym_cols<D, TIn>(Rs, s, w, i, g); }, wk, pn, tid);
}

// P_s = pn + the symmetric part of the stage cost goes to the right half, exactly symmetric; add_Q(pn, w, i, g) adds it.
// Contains the barriers it needs.
template <int D, typename AddQ>
__device__ __forceinline__ void next_value_matrix_with(float* W, AddQ&& add_Q, Cols<D>& pn, int tid) {
  const int lane = tid & 63, w = uniform(tid >> 6), i = lane & 15, g = lane >> 4;
  add_Q(pn, w, i, g);
  store_cols_T<D>(W + D, pn, w, i, g);  // (the solve ended with a barrier: the right half is free)
  lds_barrier();
  symmetrise_half<D>(W + D, tid);
  lds_barrier();
}
template <int D, typename TIn>
__device__ __forceinline__ void next_value_matrix(float* W, const TIn* Qs, Cols<D>& pn, int tid) {
  next_value_matrix_with<D>(
      W, [&](Cols<D>& m, int w, int i, int g) { add_sym_cols<D, TIn>(Qs, m, w, i, g); }, pn, tid);
}

}  // namespace ttc
