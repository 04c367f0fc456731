// The default path of ttc_lqr_solve at d = 16: the T equal factors composed by squaring (the algebra of ttc_doubling.hpp, the
// guard of ttc_squaring.hpp), from register to register, one problem to a wavefront or four.
//
// The layouts are those of a step of the recursion (ttc_tv.hpp): a matrix in the accumulator layout (lane (i, g) holds
// M[4g + v][i]) is the right operand of a product and the left operand of the transpose's.  A_e is held in it and transposed (a row
// of four entries a lane), G_e, H_e and P are symmetric.  I + G_e H_e is formed transposed, so that its inverse comes as a left
// operand.  A squaring is eight products of four matrix instructions and one inverse, a step of the recursion ten and one; what
// counts is that T factors take log2 T squarings (and the bits of T an application each, four products and an inverse).
//
// One problem to a wavefront is bound by its chain of dependent instructions (the inverse alone is half of a squaring), four by
// issue: float32 matrix instructions and the vector instructions of the inverses take turns.  Measured against the sequential product
// (solve_small_kernel), float32, us a call: 16384 problems T = 8 140 -> 69, T = 31 419 -> 119; 2000 problems T = 19 81 -> 26; P_0 off by
// 1.6e-6 for 1.9e-5 at T = 8, 8.9e-6 for 1.6e-5 at T = 31 (the worst of 4096 problems).
#pragma once
#include "ttc_small_kernel.hpp"

namespace ttc {

// The guard, on max |I + G_e H_e| and max |I + P G_e| over the wavefront's problems (ttc_squaring.hpp has what it rests on): what is large
// in the first squaring is cheap control, which loses digits, and is left to the recursion (float32 from 8 on: ordinary problems stay below 7,
// T = 8 with R scaled by 0.1 7.6e-6 by squaring, 1.5e-6 by the recursion), which together with the attempt costs less than the sequential
// product did, whose guard gives most of these up as well (product / this, us a call: R scaled by 0.1, 16384 problems T = 8 164 / 150, T = 33 526 /
// 505, 2000 problems 47 / 33 and 143 / 100; by 0.01 the same, 2000 problems 37 / 33 and 107 / 100); growth that comes later is that of an unstable open loop, and the power reached is then applied as often as needed
// instead of squared again.
static constexpr float SQUARE16_FIRST_F32 = 8.f, SQUARE16_FIRST_BF16 = 24.f, SQUARE16_LATE = 256.f, SQUARE16_STOP = 16.f;
// Where P starts from a terminal cost of its own, P G_e is a product of matrices that know nothing of each other, and elimination in order
// loses more: pivots are searched from 12 on, or behind one below PIVOT16_FIRST (Q_T = 10 Q, T = 2 6.8e-5 with the limits above, 2.2e-6 so;
// the sequential product 1.4e-5).  Without a running cost I + G_e H_e is the identity however fast G_e grows: there max |Q_T| max |G_e| is
// looked at in its place, and from 64 on, as predicted, the power is kept.
static constexpr float SQUARE16_QT_IN_ORDER = 12.f, SQUARE16_QT_STOP = 64.f;
// Elimination is in order up to this; above it, and where a late one meets a pivot below PIVOT16_LATE (one in two thousand problems at
// T = 31, rho(A) = 1.1), it searches pivots.  In the first squaring a small pivot means a stage cost that is not semidefinite.
static constexpr float SQUARE16_IN_ORDER = 24.f, PIVOT16_FIRST = 0.25f, PIVOT16_LATE = 0.0625f;
// The limit on the diagonal of the inverses of I + G_e H_e and I + P G_e.  Stage costs that are not semidefinite lose digits where an
// eigenvalue of such a matrix comes near 0, on its way below, and its inverse becomes large; with semidefinite ones it has eigenvalues
// within (0, 1].  The diagonal, as the other entries depend on the units of the states.  The algorithm in float32 against float64: semidefinite
// costs (of low rank, in units far apart, unstable, cheap control: 1800 problems) up to 1.47; 14000 problems with eigenvalues of Q below 0,
// T = 3 to 32, kept under a limit of 2: one off by more than 1e-4 and ten times what the recursion with general solves is (1.1 times that),
// of 3: six, without a limit 100 times as many (one of two, Q = I with one eigenvalue of -1, T = 4: up to 7.8e-3).
static constexpr float SQUARE16_INVERSE = 2.f;

// Four registers a lane of four matrices (x[q], lane group g: the entries 4g + v of a row) to a row of sixteen per lane, matrix q in
// lane group q, and back: registers and lane groups change places, four swaps for each v.
__device__ __forceinline__ void rows_of_quad(const floatx4 (&x)[4], float (&a)[16]) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const auto e = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[0][v]), __float_as_uint(x[2][v]), false, false);
    const auto o = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[1][v]), __float_as_uint(x[3][v]), false, false);
    const auto l = __builtin_amdgcn_permlane16_swap(e[0], o[0], false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(e[1], o[1], false, false);
    a[v] = __uint_as_float(l[0]);
    a[4 + v] = __uint_as_float(l[1]);
    a[8 + v] = __uint_as_float(h[0]);
    a[12 + v] = __uint_as_float(h[1]);
  }
}
__device__ __forceinline__ void quad_of_rows(const float (&a)[16], floatx4 (&x)[4]) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const auto e = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[v]), __float_as_uint(a[8 + v]), false, false);
    const auto o = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[4 + v]), __float_as_uint(a[12 + v]), false, false);
    const auto l = __builtin_amdgcn_permlane16_swap(e[0], o[0], false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(e[1], o[1], false, false);
    x[0][v] = __uint_as_float(l[0]);
    x[1][v] = __uint_as_float(l[1]);
    x[2][v] = __uint_as_float(h[0]);
    x[3][v] = __uint_as_float(h[1]);
  }
}

// The inverses of the wavefront's matrices, elimination in order: lane (i, g) holds M[i][4g .. 4g+3] and ends with the same entries of
// the inverse.  Returns, uniformly, whether a pivot of any of them was not above piv_min and finite.
template <int PPW, bool SYMMETRIC>
__device__ __forceinline__ bool invert16(floatx4 (&x)[PPW], float (*Wm)[16 * Cfg<16>::PITCH], int lane, float piv_min) {
  if constexpr (PPW == 1) {
    return (SYMMETRIC ? invert_spread16(x[0], lane, piv_min) : invert_spread16(x[0], Wm[0], Cfg<16>::PITCH, lane, piv_min)) != 0;
  } else {
    float a[16];
    rows_of_quad(x, a);
    const int bad = invert_regs16(a, piv_min);
    quad_of_rows(a, x);
    return __any(bad);
  }
}

// x summed over the four lane groups
__device__ __forceinline__ float sum_groups(float x) {
  const unsigned u = __float_as_uint(x);
  const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const float y = __uint_as_float(h[0]) + __uint_as_float(h[1]);
  const unsigned t = __float_as_uint(y);
  const auto q = __builtin_amdgcn_permlane16_swap(t, t, false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// Whether A, its columns divided by their diagonal entries, is within 1/sqrt(2) of the identity in the Frobenius norm: then it is not
// singular, which else takes a factorisation to know (a singular A is reported, although nothing here divides by A).  False for
// anything that overflows, vanishes or is not finite on the way.
__device__ __forceinline__ bool near_diagonal16(const floatx4& A, int i, int g) {
  float sq = 0.f, on = 0.f;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    on = 4 * g + v == i ? A[v] : on;
    sq = __builtin_fmaf(A[v], A[v], sq);
  }
  sq = sum_groups(sq);
  on = sum_groups(on);
  const float e = sum16(sq / (on * on));
  return __all(e < 16.5f);
}

// The inverses of matrices of any kind, with a search for pivots, through LDS; the solve is a function of its own, as few problems need
// it.  Returns, uniformly, whether one broke down.
template <int PPW>
__device__ __attribute__((noinline)) bool solve_rows16_called(float (*Wm)[16 * Cfg<16>::PITCH], int lane) {
  return __any(solve_rows16<true>(in_lds(Wm)[(lane >> 4) & (PPW - 1)], lane));
}
template <int PPW>
__device__ __forceinline__ bool invert_pivoted16(floatx4 (&x)[PPW], float (*Wm)[16 * Cfg<16>::PITCH], int lane) {
  using C = Cfg<16>;
  const int i = lane & 15, g = lane >> 4;
#pragma unroll
  for (int q = 0; q < PPW; ++q) {
    float* const row = Wm[q] + i * C::PITCH + 4 * g;
    *reinterpret_cast<floatx4*>(row) = x[q];
    floatx4 e;
#pragma unroll
    for (int v = 0; v < 4; ++v) e[v] = 4 * g + v == i ? 1.f : 0.f;
    *reinterpret_cast<floatx4*>(row + 16) = e;
  }
  wave_lds_sync();
  const bool bad = solve_rows16_called<PPW>(Wm, lane);
#pragma unroll
  for (int q = 0; q < PPW; ++q) x[q] = *reinterpret_cast<const floatx4*>(Wm[q] + i * C::PITCH + 4 * g + 16);
  wave_lds_sync();
  return bad;
}

// Whether a diagonal entry of a symmetric matrix is negative, which it is in no semidefinite one.
template <int PPW>
__device__ __forceinline__ bool negative_diagonal16(const floatx4 (&H)[PPW], int i, int g) {
  float least = 0.f;
#pragma unroll
  for (int q = 0; q < PPW; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) least = 4 * g + v == i ? __builtin_fminf(least, H[q][v]) : least;
  return __any(least < 0.f);
}

// Whether a diagonal entry is above the limit in magnitude, or not a number; first of all the entries, which in most problems are below.
template <int PPW>
__device__ __forceinline__ bool large_diagonal16(const floatx4 (&M)[PPW], float limit, int i, int g) {
  float all = 0.f, on = 0.f;
#pragma unroll
  for (int q = 0; q < PPW; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) all = __builtin_elementwise_maximum(all, __builtin_fabsf(M[q][v]));
  if (!__any(!(all <= limit))) return false;
#pragma unroll
  for (int q = 0; q < PPW; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) on = 4 * g + v == i ? __builtin_elementwise_maximum(on, __builtin_fabsf(M[q][v])) : on;
  return __any(!(on <= limit));
}

template <int PPW>
__device__ __forceinline__ void identity16(floatx4 (&M)[PPW], int i, int g) {
#pragma unroll
  for (int q = 0; q < PPW; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) M[q][v] = 4 * g + v == i ? 1.f : 0.f;
}

// The largest magnitude of all entries, NaN on top.
template <int PPW>
__device__ __forceinline__ float largest16(const floatx4 (&M)[PPW]) {
  uint32_t big = 0;
#pragma unroll
  for (int q = 0; q < PPW; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const uint32_t b = __float_as_uint(M[q][v]) & 0x7FFFFFFFu;
      big = b > big ? b : big;
    }
  return __uint_as_float(wave_max_u32(big));
}

// What squaring cannot do, by the recursion (recursion) or by the sequential product of solve_small_kernel, which also is for what breaks
// the recursion down; a function of its own, as few problems need it.
template <typename TIn, int PPW>
__device__ __attribute__((noinline)) void solve_otherwise16(const SolveArgs args, long long quad, bool recursion,
                                                            float (*Wm_)[16 * Cfg<16>::PITCH], float* s_red_, float (*s_x0_)[16]) {
  const SolveArgs p = called_args(args);
  quad = uniform64(quad);
  float(*const Wm)[16 * Cfg<16>::PITCH] = in_lds(Wm_);
  float* const s_red = in_lds(s_red_);
  float(*const s_x0)[16] = in_lds(s_x0_);
  if (recursion) {
    long long prob[PPW];
    bool valid[PPW];
    const TIn *Ap[PPW], *Bp[PPW], *Qp[PPW], *Rp[PPW], *PTp[PPW];
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
      valid[q] = quad * PPW + q < p.n;
      prob[q] = valid[q] ? quad * PPW + q : p.n - 1;
      Ap[q] = reinterpret_cast<const TIn*>(p.A) + prob[q] * p.sA;
      Bp[q] = reinterpret_cast<const TIn*>(p.B) + prob[q] * p.sB;
      Qp[q] = reinterpret_cast<const TIn*>(p.Q) + prob[q] * p.sQ;
      Rp[q] = reinterpret_cast<const TIn*>(p.R) + prob[q] * p.sR;
      PTp[q] = p.QT ? reinterpret_cast<const TIn*>(p.QT) + prob[q] * p.sQT : Qp[q];
    }
    if (!riccati_quad<TIn, PPW>(Wm, p, prob, valid, p.T, Ap, Bp, Qp, Rp, PTp, 0, 0, 0, 0, 2, threadIdx.x + opaque_zero())) return;
    __syncthreads();
  }
  solve_small_quad<TIn, PPW>(p, quad, Wm, s_red, s_x0);
}

// The wavefront's problems by squaring; 0, or why it was given up: 1 to the recursion, 2 to the product.
// OWN_QT: Q_T is a matrix of its own.  A template argument, as the registers of what only such problems need cost the others 3 % (16384
// problems, T = 8, 68.4 -> 70.1 us); P is read and started under the argument da.p_from_qt all the same, without which the other instance
// spills 15 registers for 11 (69.8).
template <typename TIn, int PPW, bool OWN_QT>
__device__ __forceinline__ int square_quad16(const DoublingArgs& da, long long quad, float (*Wm)[16 * Cfg<16>::PITCH]) {
  using C = Cfg<16>;
  constexpr float FIRST = sizeof(TIn) == 4 ? SQUARE16_FIRST_F32 : SQUARE16_FIRST_BF16;
  const SolveArgs& p = da.s;
  const int lane = (threadIdx.x + opaque_zero()) & 63, i = lane & 15, g = lane >> 4;
  long long prob[PPW];  // a ragged last quad repeats the last problem; only valid ones are written out
  bool valid[PPW];
  const TIn *Ap[PPW], *Bp[PPW], *Qp[PPW], *Rp[PPW];
#pragma unroll
  for (int q = 0; q < PPW; ++q) {
    valid[q] = quad * PPW + q < p.n;
    prob[q] = valid[q] ? quad * PPW + q : p.n - 1;
    Ap[q] = reinterpret_cast<const TIn*>(p.A) + prob[q] * p.sA;
    Bp[q] = reinterpret_cast<const TIn*>(p.B) + prob[q] * p.sB;
    Qp[q] = reinterpret_cast<const TIn*>(p.Q) + prob[q] * p.sQ;
    Rp[q] = reinterpret_cast<const TIn*>(p.R) + prob[q] * p.sR;
  }
  // ---- set-up: A and its transpose, G = B R^{-1} B^T, H = Q
  floatx4 A[PPW], AT[PPW], G[PPW], H[PPW], P[PPW], x[PPW], n[PPW];
  {
    floatx4 BT[PPW], R[PPW], X[PPW], t[PPW];
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
      A[q] = load_acc16<TIn>(Ap[q], i, g);
      AT[q] = load_accT16<TIn>(Ap[q], i, g);
      BT[q] = load_accT16<TIn>(Bp[q], i, g);
      R[q] = 0.5f * (load_acc16<TIn>(Rp[q], i, g) + load_accT16<TIn>(Rp[q], i, g));
      H[q] = 0.5f * (load_acc16<TIn>(Qp[q], i, g) + load_accT16<TIn>(Qp[q], i, g));
      if (da.p_from_qt) {
        const TIn* QTp = reinterpret_cast<const TIn*>(p.QT) + prob[q] * p.sQT;
        P[q] = 0.5f * (load_acc16<TIn>(QTp, i, g) + load_accT16<TIn>(QTp, i, g));
      }
    }
    if (negative_diagonal16<PPW>(H, i, g)) return 2;  // squaring loses all digits where a stage cost is not semidefinite
    bool regular = true;
#pragma unroll
    for (int q = 0; q < PPW; ++q) regular = near_diagonal16(A[q], i, g) && regular;
    if (!regular) {
#pragma unroll
      for (int q = 0; q < PPW; ++q) x[q] = A[q];
      if (invert_pivoted16<PPW>(x, Wm, lane)) return 2;
    }
#pragma unroll
    for (int q = 0; q < PPW; ++q) x[q] = R[q];
    if (invert16<PPW, true>(x, Wm, lane, 0.f)) return 2;
    zero16<PPW>(X);
    mul16<PPW>(X, x, BT);  // R^{-1} B^T, refined once
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
      t[q] = BT[q];
      R[q] = -R[q];
    }
    mul16<PPW>(t, R, X);
    mul16<PPW>(X, x, t);
    zero16<PPW>(G);
    mul16<PPW>(G, BT, X);
    symmetrise16<PPW>(G, i, g);
    if (OWN_QT && da.m && !(da.m & 1)) {
      // A terminal cost over its limit with the first G_e already goes at once, not behind the squarings ahead of its application.  (By its
      // size beside Q's, as before, one beside a small running cost went too, to the recursion: Q = 0, T = 8, 16384 problems 153 us, by
      // squaring 90; T = 33 520, 134.)
      identity16<PPW>(n, i, g);
      mul16<PPW>(n, G, P);
      if (!(largest16<PPW>(n) <= SQUARE16_LATE)) return 1;
    }
  }
  // ---- P_1 by binary powering of the one-step map.  A turn either applies e to P or squares it: both begin with the inverse of a
  // matrix I + (symmetric)(symmetric), formed transposed.
  bool have_p = da.p_from_qt != 0;
  bool bit_done = false;  // P has had the current bit of m
  bool stay = false;      // e is not squared any further, but applied once for each factor of it that is left
  float up_prev = 0.f;    // max |I + G_e H_e| - 1 (H = 0: max |Q_T| max |G_e|) of the squaring before, 0 before the first
  float qt_max = 0.f;     // max |Q_T| if H = 0, or else 0
  if constexpr (OWN_QT) qt_max = largest16<PPW>(H) == 0.f ? largest16<PPW>(P) : 0.f;
  for (int m = da.m; m;) {
    bool apply = false;
    if (!bit_done && ((m & 1) || stay)) {
      apply = have_p;
      if (!have_p) {  // f_e(0) = H_e
        have_p = true;
#pragma unroll
        for (int q = 0; q < PPW; ++q) P[q] = H[q];
      }
    }
    if (!apply) {
      bit_done = false;
      if (stay) {
        --m;
        continue;
      }
      m >>= 1;
      if (!m) break;
    }
    const bool only_H = !apply && m == 1 && !have_p;  // the last squaring, and P is still 0: A and G of the square are not needed
    auto form = [&] {
      identity16<PPW>(n, i, g);
      if (apply) mul16<PPW>(n, G, P);  // (I + P G)^T
      else mul16<PPW>(n, H, G);        // (I + G H)^T
    };
    form();
    const float mu = largest16<PPW>(n);
    const float up = (OWN_QT && qt_max != 0.f && !apply) ? qt_max * largest16<PPW>(G) : mu - 1.f;
    const bool early = !apply && up_prev == 0.f;
    const bool own = OWN_QT && apply;
    if (!(mu <= (early ? FIRST : SQUARE16_LATE))) return negative_diagonal16<PPW>(H, i, g) ? 2 : 1;
    if (!apply) {
      // mu - 1 has grown by r, and the square of e will make it grow by r^2 at least
      const float stop = qt_max != 0.f ? SQUARE16_QT_STOP : SQUARE16_STOP;
      if (!only_H && up_prev != 0.f && up > 1.f && up > 2.f * up_prev && up * up * up > stop * up_prev * up_prev) {
        stay = true;
        m *= 2;
        continue;
      }
      up_prev = up;
    }
    bool pivoted = mu > (own ? SQUARE16_QT_IN_ORDER : SQUARE16_IN_ORDER);
    if (!pivoted && invert16<PPW, false>(n, Wm, lane, early || own ? PIVOT16_FIRST : PIVOT16_LATE)) {
      if (early) return 2;
      if (negative_diagonal16<PPW>(H, i, g)) return 2;
      form();
      pivoted = true;
    }
    if (__builtin_expect(pivoted, 0) && invert_pivoted16<PPW>(n, Wm, lane)) return 2;
    if (large_diagonal16<PPW>(n, SQUARE16_INVERSE, i, g)) return 2;
    zero16<PPW>(x);
    if (apply) {
      mul16<PPW>(x, P, A);
      floatx4 t[PPW];
      zero16<PPW>(t);
      mul16<PPW>(t, n, x);  // M P A
#pragma unroll
      for (int q = 0; q < PPW; ++q) P[q] = H[q];
      mul16<PPW>(P, A, t);  // H_e + A_e^T (I + P G_e)^{-1} P A_e
      symmetrise16<PPW>(P, i, g);
      if (stay) --m;
      else bit_done = true;
      continue;
    }
    mul16<PPW>(x, n, A);  // M A
    floatx4 V[PPW];
    if (!only_H) {
      floatx4 Y[PPW], Z[PPW];
      zero16<PPW>(Y);
      mul16<PPW>(Y, n, G);  // M G, symmetric
      zero16<PPW>(Z);
      mul16<PPW>(Z, Y, AT);  // M G A^T
      mul16<PPW>(G, AT, Z);  // G + A M G A^T
      zero16<PPW>(Y);
      mul16<PPW>(Y, AT, x);  // A M A
      zero16<PPW>(V);
      mul16<PPW>(V, H, x);  // H M A
      mul16<PPW>(H, A, V);  // H + A^T H M A
#pragma unroll
      for (int q = 0; q < PPW; ++q) {
        A[q] = Y[q];
        *reinterpret_cast<floatx4*>(Wm[q] + i * C::PITCH + 4 * g) = Y[q];  // the transpose, row-major
      }
      wave_lds_sync();
#pragma unroll
      for (int q = 0; q < PPW; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) AT[q][v] = Wm[q][(4 * g + v) * C::PITCH + i];
      wave_lds_sync();
    } else {
      zero16<PPW>(V);
      mul16<PPW>(V, H, x);
      mul16<PPW>(H, A, V);
    }
  }
  if (!have_p) return 2;  // (not reached: m >= 1, or P starts at Q_T)
  // ---- last step, with the problem's own matrices: as printed
  symmetrise16<PPW>(P, i, g);
  floatx4 Wk[PPW], pn[PPW];
  {
    floatx4 B[PPW], S[PPW], Si[PPW];
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
      A[q] = load_acc16<TIn>(Ap[q], i, g);
      B[q] = load_acc16<TIn>(Bp[q], i, g);
    }
    const int bad = riccati_step16<PPW, true>(Wm, P, A, B,
                                        [&](int q) { return 0.5f * (load_acc16<TIn>(Rp[q], i, g) + load_accT16<TIn>(Rp[q], i, g)); },
                                        [] {}, Wk, pn, S, Si, lane);
    if (__any(bad)) return 2;
  }
  symmetrise16<PPW>(pn, i, g);
  wave_lds_sync();
  const int fine[PPW] = {};
  emit_quad16<TIn, PPW>(Wm, p, prob, valid, Qp, pn, Wk, fine, 0, lane);
  return 0;
}

template <typename TIn, int PPW, bool OWN_QT>
__global__ void __launch_bounds__(64, PPW == 4 ? 2 : 3) squaring16_kernel(const DoublingArgs da) {
  constexpr int D = 16;
  using C = Cfg<D>;
  static_assert(PPW == 1 || PPW == 4, "one problem or four per wavefront");
  __shared__ __attribute__((aligned(16))) float Wm[PPW][D * C::PITCH];
  __shared__ float s_red[C::NW];
  __shared__ __attribute__((aligned(16))) float s_x0[PPW][D];
  const long long nquads = (da.s.n + PPW - 1) / PPW;
  for (long long quad = blockIdx.x; quad < nquads; quad += gridDim.x) {
    const int why = uniform(square_quad16<TIn, PPW, OWN_QT>(da, quad, Wm));
    if (__builtin_expect(why != 0, 0)) {
      __syncthreads();
      solve_otherwise16<TIn, PPW>(da.s, quad, why == 1, Wm, s_red, s_x0);
      __syncthreads();
    }
  }
}

}  // namespace ttc
