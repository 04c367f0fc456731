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
// P (A - E), A^T Y = E Y + (A - E)^T Y) costs one addition in the accumulator and leaves the product with what is small where the
// dynamics are near the identity; gradients of 8 steps at d = 64 are off by 0.7 times what float32 products gave (24 steps: 0.6).
//
// Measured, T = 8, float32, float32 products -> split: roll-out d = 64, 4096 problems 1.36 -> 0.95 ms, d = 32, 8192 problems 0.54 ->
// 0.46, d = 128, 1024 problems 2.77 -> 1.71; backward pass d = 64, 8192 problems 2.91 -> 2.21; ttc_lqr_solve_tv d = 64, 1024
// problems 0.36 -> 0.28.  At d = 64 a step of one problem alone takes 24 thousand cycles (28), of which the dense solve is 13:
// what is left is its serial chain, hidden as far as three workgroups a compute unit allow.
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
// Of a row-major matrix in memory, the signs (1 or -1) of the diagonal entries of a lane's columns; m -= diag(e).
template <int D, typename TIn>
__device__ __forceinline__ void load_diagonal_signs(const TIn* M, float (&e)[Cfg<D>::RB], int w, int i) {
#pragma unroll
  for (int k = 0; k < Cfg<D>::RB; ++k)
    e[k] = __builtin_copysignf(1.f, ld1<TIn>(M, (long)(16 * (Cfg<D>::RB * w + k) + i) * (D + 1)));
}
template <int D>
__device__ __forceinline__ void subtract_diagonal(Cols<D>& m, const float (&e)[Cfg<D>::RB], int w, int i, int g) {
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int k = 0; k < Cfg<D>::RB; ++k)
#pragma unroll
      for (int v = 0; v < 4; ++v) m[r][k][v] -= (r == Cfg<D>::RB * w + k && 4 * g + v == i) ? e[k] : 0.f;
}
// from a row-major matrix in memory: a row of 16 lanes reads 16 consecutive elements
template <int D, typename TIn>
__device__ __forceinline__ void load_cols(const TIn* M, Cols<D>& m, int w, int i, int g) {
  const unsigned o = (unsigned)(4 * g * D + 16 * Cfg<D>::RB * w + i);
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int k = 0; k < Cfg<D>::RB; ++k) m[r][k][v] = ld1<TIn>(M, o + (unsigned)((16 * r + v) * D + 16 * k));
}
// its transpose (a lane's four entries are consecutive elements)
template <int D, typename TIn>
__device__ __forceinline__ void load_cols_T(const TIn* M, Cols<D>& m, int w, int i, int g) {
  const unsigned o = (unsigned)((16 * Cfg<D>::RB * w + i) * D + 4 * g);
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int k = 0; k < Cfg<D>::RB; ++k) m[r][k] = ld4<TIn>(M, o + (unsigned)(16 * k * D + 16 * r));
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
  Cols<D> t;
  load_cols<D, TIn>(M, t, w, i, g);
  const unsigned o = (unsigned)((16 * Cfg<D>::RB * w + i) * D + 4 * g);
#pragma unroll
  for (int r = 0; r < D / 16; ++r)
#pragma unroll
    for (int k = 0; k < Cfg<D>::RB; ++k) m[r][k] += 0.5f * (t[r][k] + ld4<TIn>(M, o + (unsigned)(16 * k * D + 16 * r)));
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
// or any whose elimination in order meets pivots above piv_min only: block Gauss-Jordan with 16 x 16 pivot blocks and no pivot search.  Per block p, the wavefront that owns its columns
// inverts s[p][p] in registers and publishes that inverse and the rest of the column, negated, as left operands (Wp: the
// right half of the pair); every wavefront then does its own columns, U = s[p][p]^{-1} s[p][c], s[r][c] -= s[r][p] U,
// the next block's first, so that its inverse is formed and published under the others' updates: one workgroup barrier
// per block, no right operand through LDS, and a serial chain of some 1500 cycles per 16 columns (the pivoted panels of
// lds_solve: about 5000).
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
    bad |= invert_spread16(inv, lane, piv_min);
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
          column(x, s, IntC<kn>{}, p);
          publish(IntC<kn>{}, buf ^ 1);
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
    bad |= invert_spread16(s[0][k], lane, piv_min);
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
        column(x, IntC<kn>{}, false);
        publish(IntC<kn>{}, buf ^ 1);
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

// One backward step of Prop. 3.1 with the matrices of one step.  On entry the right half of the pair holds P_{s+1}
// (symmetric, visible) and the left half is free; on exit, by columns, wk = S^{-1} B^T P A = -K_s, S = R + B^T P B, and
// pn = A^T P A - (B^T P A)^T wk, which is P_s up to the stage cost.  Six products and one unpivoted solve (S is positive
// definite).  Returns the solve's breakdown flag.  Other wavefronts may still be reading the left half on return.
// add_R(s, w, i, g) adds the symmetric part of R to s.
template <int D, typename TIn, typename AddR>
__device__ __forceinline__ int riccati_step_with(Pair<D>& W, const TIn* As, const TIn* Bs, AddR&& add_R, Cols<D>& wk,
                                                 Cols<D>& pn, int tid) {
  using C = Cfg<D>;
  tid += opaque_zero();
  const int lane = tid & 63, w = uniform(tid >> 6), i = lane & 15, g = lane >> 4;
  float* const WL = W;
  float* const WR = W + D;
  if constexpr (D == 16) {  // one tile: half of a float16 instruction's depth would be empty
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
    using Split = SplitCols<D, C::RB>;
    constexpr int L = 0, R = 1;  // the halves
    float* const signs = W + D * C::PITCH;
    float e[C::RB];
    Cols<D> s;
    {
      Split a;
      {
        Split b;
        Cols<D> t;
        {
          Cols<D> bc;
          Split p;
          load_cols<D, TIn>(Bs, bc, w, i, g);
          load_cols<D, TIn>(As, t, w, i, g);
          load_diagonal_signs<D, TIn>(As, e, w, i);
          zero_cols<D>(s);
          add_R(s, w, i, g);
          TTC_SCHED_BARRIER();  // the step's reads are all under way
          // P is symmetric: a lane's four entries of a column are four consecutive ones of its row
#pragma unroll
          for (int r = 0; r < C::NT; ++r)
#pragma unroll
            for (int k = 0; k < C::RB; ++k)
              pn[r][k] = *reinterpret_cast<const floatx4*>(WR + (16 * (C::RB * w + k) + i) * C::PITCH + 16 * r + 4 * g);
          split_cols<D, C::RB>(pn, p);
          lds_barrier();  // every wavefront has read its columns of P
          store_split_T<D>(W, R, p, w, i, g);  // P
          split_cols<D, C::RB>(bc, b);
          store_split_T<D>(W, L, b, w, i, g);  // B^T
        }
        subtract_diagonal<D>(t, e, w, i, g);
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
#pragma unroll
      for (int r = 0; r < C::NT; ++r)
#pragma unroll
        for (int k = 0; k < C::RB; ++k) pn[r][k] = pn[r][k] * e[k];
      gemm_split<D, C::RB, true>(pn, W, R, a, i, g);  // P A = P E + P (A - E)
      split_cols<D, C::RB>(pn, pa);
      gemm_split<D, C::RB>(wk, W, L, pa, i, g);  // F = B^T P A
      Split f;
      split_cols<D, C::RB>(wk, f);
      lds_barrier();                           // P and B^T are no longer read
      store_split_T<D>(W, R, a, w, i, g);  // (A - E)^T
      store_split_T<D>(W, L, f, w, i, g);  // F^T
      lds_barrier();
#pragma unroll
      for (int r = 0; r < C::NT; ++r) {
        const floatx4 er = *reinterpret_cast<const floatx4*>(signs + 16 * r + 4 * g);
#pragma unroll
        for (int k = 0; k < C::RB; ++k) pn[r][k] = pn[r][k] * er;
      }
      gemm_split<D, C::RB, true>(pn, W, R, pa, i, g);  // A^T P A = E P A + (A - E)^T P A
    }
    lds_barrier();
    const int flag = solve_cols<D, C::RB>(WR, s, wk, w, lane);  // W = S^{-1} F
    Split x;
    split_cols<D, C::RB>(wk, x);
    gemm_split<D, C::RB, true, -1>(pn, W, L, x, i, g);  // - F^T W
    return flag;
  }
}

template <int D, typename TIn>
__device__ __forceinline__ int riccati_step(Pair<D>& W, const TIn* As, const TIn* Bs, const TIn* Rs, Cols<D>& wk, Cols<D>& pn,
                                            int tid) {
  return riccati_step_with<D, TIn>(
      W, As, Bs, [&](Cols<D>& s, int w, int i, int g) { add_sym_cols<D, TIn>(Rs, s, w, i, g); }, wk, pn, tid);
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
