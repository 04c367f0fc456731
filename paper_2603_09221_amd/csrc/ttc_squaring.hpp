// The default path of ttc_lqr_solve for longer horizons at d >= 32: time-invariant parameters make the T factors of
// Thm 3.3 equal, so their product is formed by squaring (the algebra of ttc_doubling.hpp), with the element on chip.
//
// The sequential product costs four products per factor and a pivoted solve per group of three or so, whatever T; a
// squaring costs eight products and one solve and doubles the number of factors, and on ordinary problems it is several
// times more accurate (no A^{-1}, no accumulated pair).  Its weak side is accuracy when control is cheap: I + G_e H_e is
// large from the first squaring on, and the composition loses digits in proportion.  The kernel watches
// mu = max |I + G_e H_e| (and max |I + P G_e|) and gives up a problem that passes the limits below.
//
// Measured (float32, d = 32, 64, 128, T = 8..64; errors against float64, product: the grouped product's):
//   ordinary problems, rho(A) 0.5..1.2          mu below 7                 1e-6..4e-6    (product 5e-6..1e-5)
//   R scaled by 0.1 / 0.03 / 0.01               mu 15 / 40 / 120           1e-5 / 2e-5 / 7e-5, in the first squaring already
//   rho(A) = 1.2, 1.3, R scaled by 1..100       mu 3..200, growing late    3e-6..8e-6    (product 2e-6..1e-5)
//   Q_T = 10 Q .. 1000 Q                        max |I + Q_T G| 15..2000   2e-6..6e-6    (product 2e-6..1e-5)
// So a large mu means lost digits in the first squaring, and there alone: p.growth_limit is the limit there, 16 for float32
// inputs (errors of 1e-5, as the product's) and 64 for bfloat16 ones, whose product in groups of five is at 1e-3 by then.
// Growth that comes later is that of an unstable open loop, whose pair (G_e, H_e) outgrows what the feedback needs
// (LATE_LIMIT); a squaring that would run into it is not done, the power reached is applied as often as there are factors
// of it left.  A terminal cost of its own meets its own limit (da.qt_limit) once, when it is first used.
//
// A problem given up is marked in its u_0 and solved by solve_handed_kernel, launched behind this one: one over a limit by
// the recursion of Prop. 3.1 in its printed form, and by the sequential product if R + B^T P B is not positive definite there
// (a stage cost that is not semidefinite, which squaring loses all digits on); one with a small pivot, a singular A or an R
// that is not positive definite by the product at once, whose reports it thereby gets.
//
// Where things live.  A_e, G_e and H_e are row blocks in registers (the A operand of a product), across the dense solves, as
// solve_kernel's constants are; LDS holds the pair a product or solve works on; the one workspace slot of the workgroup
// holds P while the bits of T still have squarings between them (never for T a power of two).  The last step is the printed
// one (riccati_step), which needs nothing but P_1 and the problem's own matrices.
#pragma once
#include "ttc_doubling.hpp"
#include "ttc_tv.hpp"

namespace ttc {

// rows[rb][k] += the wavefront's rows of the matrix in the LDS half Wh
template <int D>
__device__ __forceinline__ void add_aop_lds(const float* Wh, float (&rows)[Cfg<D>::RB][Cfg<D>::KS], int w, int i, int g) {
  using C = Cfg<D>;
  float t[C::RB][C::KS];
  load_aop_lds<D>(Wh, t, w, i, g);
#pragma unroll
  for (int rb = 0; rb < C::RB; ++rb)
#pragma unroll
    for (int k = 0; k < C::KS; ++k) rows[rb][k] += t[rb][k];
}

// Both I + G_e H_e and I + P G_e have the eigenvalues of I plus a positive semidefinite matrix.  They are not symmetric, but up
// to mu of about 30 elimination in order meets no small pivot (CPU, float64, random semidefinite pairs and the benchmark's:
// pivots of 1.1 and more; at 40 some problems in a hundred, at 120 all of them meet negative ones): the solve is solve_cols,
// without a pivot search.  Above IN_ORDER_MAX it is the pivoted lds_solve; a pivot below PIVOT_MIN (a stage cost that is not
// semidefinite, say) gives the problem up.  A is tried in order too; a pivot below PIVOT_MIN_A leaves the verdict to the pivoted
// factorisation.
static constexpr float PIVOT_MIN = 0.25f, PIVOT_MIN_A = 0.015625f, IN_ORDER_MAX = 24.f;
// The guard's limit after the first squaring, and the mu at which the coming square of e is expected and not formed.
static constexpr float LATE_LIMIT = 64.f, GROWTH_STOP = 16.f;

// One row block per wavefront at d = 128 (build.py: with two, 448 of the 512 registers hold matrices and the solves spill:
// 31.9 against 4.5 ms for 2048 problems, T = 16), two at d = 64 (2.31 against 2.84 ms for 8192 problems, T = 16).
// The recursion and the solves of the problems given up are in a kernel of their own: inlined here they spilled 345 vector and
// 107 scalar registers at d = 128 (271 and 78 without), and with R^{-1} B^T kept for a last step without R + B^T P B as well.
// The thread index is formed anew in the loop: shared with the set-up, its address arithmetic lives across the solves
// (4.15 against 4.52 ms below).
// Measured, solve_kernel / with the cold paths inlined / now: d = 128, T = 16, 2048 problems 7.01 / 4.27 / 4.15 ms, T = 64
// 35 / 5.88 / 5.74; T = 32, bfloat16 inputs 10.7 / 5.0 / 4.9; d = 64, 8192 problems, T = 8 2.14 / 1.70 / 1.65, T = 64
// 15.4 / 2.87 / 2.78; d = 32, T = 16, 16384 problems 1.6 / 0.73 / 0.69.
template <int D, typename TIn>
__global__ void __launch_bounds__(Cfg<D>::NTHR, (D <= 64 ? 2 : 1)) squaring_kernel(const DoublingArgs da) {
  using C = Cfg<D>;
  __shared__ __attribute__((aligned(16))) float W[C::PAIR];
  __shared__ __attribute__((aligned(16))) SolveScratch<D> S;
  __shared__ float s_red[C::NW];
  __shared__ float s_max[C::NW];  // per wavefront: max |I + G H| of the solve being set up
  const SolveArgs& p = da.s;
  float* const WL = W;
  float* const WR = W + D;
  float* const wsP = p.ws + (long)blockIdx.x * D * D;  // P, rows in register layout

  for (long long prob = blockIdx.x; prob < p.n; prob += gridDim.x) {
    const int tid = threadIdx.x + opaque_zero(), lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
    const TIn* Ap = reinterpret_cast<const TIn*>(p.A) + prob * p.sA;
    const TIn* Bp = reinterpret_cast<const TIn*>(p.B) + prob * p.sB;
    const TIn* Qp = reinterpret_cast<const TIn*>(p.Q) + prob * p.sQ;
    const TIn* Rp = reinterpret_cast<const TIn*>(p.R) + prob * p.sR;
    const TIn* x0p = reinterpret_cast<const TIn*>(p.x0) + prob * p.sx0;
    const TIn* QTp = da.p_from_qt ? reinterpret_cast<const TIn*>(p.QT) + prob * p.sQT : Qp;
    uint32_t give_up = 0;   // whom the problem is handed to
    bool pivoted = false;   // the dense solves search pivots, from the first large mu on
    float rA[C::RB][C::KS], rG[C::RB][C::KS], rH[C::RB][C::KS];
    floatx4 acc[C::RB][C::NT];

    // the wavefront's max |acc| for the guard; read by everyone after the next barrier
    auto publish_max = [&] {
      const float m = wave_absmax<D>(acc);
      if (lane == 0) s_max[w] = m;
    };
    auto measure = [&] {  // its maximum over the workgroup (NaN on top)
      uint32_t m = 0;
#pragma unroll
      for (int ww = 0; ww < C::NW; ++ww) {
        const uint32_t b = __float_as_uint(s_max[ww]);
        m = b > m ? b : m;
      }
      return __uint_as_float(uniform(m));
    };
    // (the word's writer is the thread that writes the first of u_0 in emit_gain)
    auto hand_over = [&](uint32_t how) {
      if (threadIdx.x == 0) reinterpret_cast<uint32_t*>(p.u0)[prob * D] = how;
      __syncthreads();  // every wavefront has left the pair
    };

    // ---- a singular A is reported, although nothing here divides by A
    load_half<D, TIn, false>(WL, Ap, tid);
    __syncthreads();
    if (solve_pair_in_order<D, false>(W, PIVOT_MIN_A, tid) && lds_factor<D>(W, S, tid)) {
      hand_over(HANDED_TO_PRODUCT);
      continue;
    }
    // ---- set-up: G = B R^{-1} B^T, A, H = Q; P = Q_T when it is a matrix of its own
    load_half<D, TIn, false>(WL, Rp, tid);
    load_half<D, TIn, false>(WR, Bp, tid);
    __syncthreads();
    symmetrise_half<D>(WL, tid);
    transpose_half<D>(WR, w, i, g);
    __syncthreads();
    if (solve_pair_in_order<D>(W, 0.f, tid)) {  // R is not positive definite
      hand_over(HANDED_TO_PRODUCT);
      continue;
    }
    {
      float c[C::RB][C::KS];
      load_aop_global<D, TIn>(Bp, c, w, i, g);
      zero_acc<D>(acc);
      gemm_acc<D>(acc, c, WR, i, g);
      store_rows<D>(WL, acc, w, i, g);
      __syncthreads();
      symmetrise_half<D>(WL, tid);  // G is symmetric up to rounding; make it exactly so
      __syncthreads();
    }
    load_aop_lds<D>(WL, rG, w, i, g);
    __syncthreads();
    load_half<D, TIn, false>(WL, Ap, tid);
    load_half<D, TIn, false>(WR, Qp, tid);
    __syncthreads();
    load_aop_lds<D>(WL, rA, w, i, g);
    symmetrise_half<D>(WR, tid);
    __syncthreads();
    load_aop_lds<D>(WR, rH, w, i, g);
    bool have_p = da.p_from_qt != 0, at_QT = have_p;  // at_QT: P is still Q_T
    if (have_p) {
      __syncthreads();
      load_half<D, TIn, false>(WR, QTp, tid);
      __syncthreads();
      symmetrise_half<D>(WR, tid);
      __syncthreads();
      float c[C::RB][C::KS];
      load_aop_lds<D>(WR, c, w, i, g);
      store_aop_ws<D>(wsP, c, tid);
    }
    __syncthreads();

    // the dense solve of the pair, whose left half's largest entry is mu.  False: a pivot below PIVOT_MIN, or none at all
    auto dense = [&](float mu) {
      pivoted = pivoted || mu > IN_ORDER_MAX;
      if (!pivoted) {
        if (solve_pair_in_order<D>(W, PIVOT_MIN, tid)) give_up = HANDED_TO_PRODUCT;
      } else {
        if (lds_solve<D>(W, S, tid)) give_up = HANDED_TO_PRODUCT;
      }
      return give_up == 0;
    };
    // [I + P G | P A] with P's rows in c, G and A as the halves hold them, then the solve: the right half becomes
    // (I + P G)^{-1} P A.  False: over the limit, or no solution
    auto mobius = [&](const float(&c)[C::RB][C::KS]) {
      eye_acc<D>(acc, w, i, g);
      gemm_acc<D>(acc, c, WL, i, g);
      publish_max();
      __syncthreads();
      const float mu = measure();
      if (!(mu <= (at_QT ? da.qt_limit : LATE_LIMIT))) {
        give_up = HANDED_TO_RECURSION;
        return false;
      }
      at_QT = false;
      store_rows<D>(WL, acc, w, i, g);
      zero_acc<D>(acc);
      gemm_acc<D>(acc, c, WR, i, g);
      __syncthreads();
      store_rows<D>(WR, acc, w, i, g);
      __syncthreads();
      return dense(mu);
    };
    // rows[rb][k] <- rH + A_e^T (the matrix in the right half), through the left half (rows may be rH itself)
    auto apply_AT = [&](float (&rows)[C::RB][C::KS]) {
      float c[C::RB][C::KS];
      store_aop_lds<D>(WL, rA, w, i, g);
      __syncthreads();
      load_aopT_lds<D>(WL, c, w, i, g);
      zero_acc<D>(acc);
      gemm_acc<D>(acc, c, WR, i, g);
      __syncthreads();
      store_rows<D>(WL, acc, w, i, g);
      __syncthreads();
      load_aop_lds<D>(WL, c, w, i, g);
#pragma unroll
      for (int rb = 0; rb < C::RB; ++rb)
#pragma unroll
        for (int k = 0; k < C::KS; ++k) rows[rb][k] = rH[rb][k] + c[rb][k];
      __syncthreads();
    };

    // ---- P_1 by binary powering of the one-step map (see ttc_doubling.hpp)
    bool p_is_H = false;  // P_1 = H_e: the last bit met no P
    float mu_prev = 0.f;  // max |I + G_e H_e| of the squaring before, 0 before the first
    bool stay = false;    // e is not squared any further, but applied once for each factor of it that is left
    for (int m = da.m; m && !give_up;) {
      const int tid = threadIdx.x + opaque_zero(), lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
      if ((m & 1) || stay) {
        if (!have_p) {
          have_p = true;
          if (m == 1) p_is_H = true;  // f_e(0) = H_e, and e is not touched again
          else store_aop_ws<D>(wsP, rH, tid);
        } else {
          float c[C::RB][C::KS];
          load_aop_ws<D>(wsP, c, tid, opaque_zero());
          store_aop_lds<D>(WL, rG, w, i, g);
          store_aop_lds<D>(WR, rA, w, i, g);
          __syncthreads();
          if (!mobius(c)) break;
          apply_AT(c);  // P <- H_e + A_e^T (I + P G_e)^{-1} P A_e
          store_aop_ws<D>(wsP, c, tid);
        }
      }
      if (stay) {
        --m;
        continue;
      }
      m >>= 1;
      if (!m) break;
      // e <- e o e
      store_aop_lds<D>(WR, rH, w, i, g);
      __syncthreads();
      eye_acc<D>(acc, w, i, g);
      gemm_acc<D>(acc, rG, WR, i, g);  // I + G H
      publish_max();
      store_rows<D>(WL, acc, w, i, g);
      __syncthreads();
      const float mu = measure();
      if (!(mu <= (mu_prev == 0.f ? p.growth_limit : LATE_LIMIT))) {
        give_up = HANDED_TO_RECURSION;
        break;
      }
      const bool only_H = m == 1 && !have_p;  // the last squaring, and P is still 0: A and G of the square are not needed
      // growth of an unstable open loop: mu - 1 has grown by r, and the square of e will make it grow by r^2 at least
      const float up = mu - 1.f, up_prev = mu_prev - 1.f;
      if (!only_H && mu_prev != 0.f && up > 1.f && up > 2.f * up_prev && up * up * up > GROWTH_STOP * up_prev * up_prev) {
        stay = true;
        m *= 2;
        continue;
      }
      mu_prev = mu;
      if (only_H) store_aop_lds<D>(WR, rA, w, i, g);
      else set_half_identity<D>(WR, tid);
      __syncthreads();
      if (!dense(mu)) break;  // right half: M = (I + G H)^{-1}, or M A
      if (only_H) {
        zero_acc<D>(acc);
        gemm_acc<D>(acc, rH, WR, i, g);  // V = H M A
        __syncthreads();
        store_rows<D>(WR, acc, w, i, g);
        apply_AT(rH);  // H' = H + A^T V
      } else {
        const int tid = threadIdx.x + opaque_zero(), lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
        float rM[C::RB][C::KS];
        load_aop_lds<D>(WR, rM, w, i, g);
        store_aop_lds<D>(WL, rA, w, i, g);
        __syncthreads();
        zero_acc<D>(acc);
        gemm_acc<D>(acc, rM, WL, i, g);  // M A
        {
          float rAT[C::RB][C::KS];
          load_aopT_lds<D>(WL, rAT, w, i, g);
          __syncthreads();
          store_rows<D>(WL, acc, w, i, g);
          __syncthreads();
          zero_acc<D>(acc);
          gemm_acc<D>(acc, rH, WL, i, g);  // V = H M A
          store_rows<D>(WR, acc, w, i, g);
          __syncthreads();
          zero_acc<D>(acc);
          gemm_acc<D>(acc, rAT, WR, i, g);  // A^T V
        }
        __syncthreads();
        store_rows<D>(WR, acc, w, i, g);
        __syncthreads();
        add_aop_lds<D>(WR, rH, w, i, g);  // H' = H + A^T V
        __syncthreads();
        store_aop_lds<D>(WR, rG, w, i, g);
        floatx4 accA[C::RB][C::NT];
        zero_acc<D>(accA);
        gemm_acc<D>(accA, rA, WL, i, g);  // A' = A M A
        __syncthreads();
        zero_acc<D>(acc);
        gemm_acc<D>(acc, rA, WR, i, g);  // A G
        __syncthreads();
        store_rows_T<D>(WR, acc, w, i, g);  // G A^T
        __syncthreads();
        zero_acc<D>(acc);
        gemm_acc<D>(acc, rM, WR, i, g);  // M G A^T
        store_rows<D>(WL, acc, w, i, g);
        __syncthreads();
        zero_acc<D>(acc);
        gemm_acc<D>(acc, rA, WL, i, g);  // A M G A^T
        store_rows<D>(WR, acc, w, i, g);  // (every wavefront is past its reads of G A^T)
        __syncthreads();
        store_rows<D>(WL, accA, w, i, g);
        __syncthreads();
        load_aop_lds<D>(WL, rA, w, i, g);
        add_aop_lds<D>(WR, rG, w, i, g);  // G' = G + A M G A^T
        __syncthreads();
      }
    }

    // ---- last step, with the problem's own matrices: as printed
    if (!give_up) {
      const int tid = threadIdx.x + opaque_zero(), lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
      if (p_is_H) {
        store_aop_lds<D>(WR, rH, w, i, g);
      } else {
        float c[C::RB][C::KS];
        load_aop_ws<D>(wsP, c, tid, opaque_zero());
        store_aop_lds<D>(WR, c, w, i, g);
      }
      __syncthreads();
      symmetrise_half<D>(WR, tid);
      __syncthreads();
      Cols<D> wk, pn;
      if (riccati_step<D, TIn>(W, Ap, Bp, Rp, wk, pn, tid)) give_up = HANDED_TO_PRODUCT;
      else emit_step<D, TIn>(W, s_red, p, prob, wk, pn, Qp, x0p, 0, tid);
    }
    if (give_up) hand_over(give_up);
  }
}

}  // namespace ttc
