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
// Where things live.  Everything is held by columns (ttc_columns.hpp), products run on split operands (ttc_split.hpp): G_e and H_e
// in float32 registers, A_e and its transpose as split registers, which are right operands as they stand and, stored, the left
// operands of each other.  I + G_e H_e is formed transposed, H_e on the left, so that the columns of its inverse are the rows of M
// as a left operand; eight products and one inverse a squaring, each product's result split where it is the next one's operand.
// The one workspace slot of the workgroup holds P while the bits of T still have squarings between them (never for T a power of
// two).  The last step is the printed one (riccati_step), which needs nothing but P_1 and the problem's own matrices.
#pragma once
#include "ttc_doubling.hpp"
#include "ttc_tv.hpp"

namespace ttc {


// The pivoted solve and factorisation, which few problems need: at d = 128 as functions of their own, as inlined their registers
// push the element of the problem into memory on every path (T = 16, 8192 problems 10.96 -> 10.71 ms); at d = 64 the call itself
// costs more (T = 8, 16384 problems 2.55 -> 3.02 ms).
template <int D>
__device__ __attribute__((noinline)) int lds_solve_called(float* W, SolveScratch<D>& S, int tid) {
  return lds_solve<D>(W, S, tid);
}
template <int D>
__device__ __attribute__((noinline)) int lds_factor_called(float* W, SolveScratch<D>& S, int tid) {
  return lds_factor<D>(W, S, tid);
}
template <int D>
__device__ __forceinline__ int lds_solve_aside(float* W, SolveScratch<D>& S, int tid) {
  if constexpr (D == 128) return lds_solve_called<D>(W, S, tid);
  else return lds_solve<D>(W, S, tid);
}
template <int D>
__device__ __forceinline__ int lds_factor_aside(float* W, SolveScratch<D>& S, int tid) {
  if constexpr (D == 128) return lds_factor_called<D>(W, S, tid);
  else return lds_factor<D>(W, S, tid);
}

// f <- s^{-1} f for a symmetric positive definite s, fs being f in split form, through the right half of the pair (s is lost).  At
// d = 128 by the inverse and a product: right-hand sides carried along double the float32 matrix instructions of an elimination
// (73 thousand cycles, against 44 for an inverse and 5 for the product); at d = 64 both take 13 thousand.  For R alone, where
// nothing is subtracted from what it gives: errors grow with R's condition number as a solve's do (T = 16, condition 1e4, 1e6: P_0 3.5e-6,
// 1.4e-4; float32 products and a pivoted solve 7.2e-6, 3.1e-4; the recursion 2.4e-6, 1.3e-4).  In a step of the recursion, whose value
// matrix is a difference, an explicit inverse loses too much (cost ratio 1e4: 8e-3 in P_0 for 1e-3).
// Returns the breakdown flag; the right half is free.
template <int D>
__device__ __forceinline__ int invert_or_solve(Pair<D>& W, Cols<D>& s, Cols<D>& f, const SplitCols<D, Cfg<D>::RB>& fs, int w, int lane,
                                               int i, int g) {
  using C = Cfg<D>;
  if constexpr (D == 128) {
    const int flag = invert_cols<D>(W + D, s, w, lane, 0.f);
    SplitCols<D, C::RB> t;
    split_cols<D, C::RB>(s, t);
    store_split_T<D>(W, 1, t, w, i, g);
    lds_barrier();
    gemm_split<D, C::RB>(f, W, 1, fs, i, g);
    lds_barrier();
    return flag;
  } else {
    return solve_cols<D, C::RB>(W + D, s, f, w, lane);
  }
}

// Both I + G_e H_e and I + P G_e have the eigenvalues of I plus a positive semidefinite matrix.  They are not symmetric, but up
// to mu of about 30 elimination in order meets no small pivot (CPU, float64, random semidefinite pairs and the benchmark's:
// pivots of 1.1 and more; at 40 some problems in a hundred, at 120 all of them meet negative ones): the solve is by columns,
// without a pivot search.  Above IN_ORDER_MAX it is the pivoted lds_solve; a pivot below PIVOT_MIN (a stage cost that is not
// semidefinite, say) gives the problem up.  A is tried in order too; a pivot below PIVOT_MIN_A leaves the verdict to the pivoted
// factorisation.
static constexpr float PIVOT_MIN = 0.25f, PIVOT_MIN_A = 0.015625f, IN_ORDER_MAX = 24.f;
// The guard's limit after the first squaring, and the mu at which the coming square of e is expected and not formed.
static constexpr float LATE_LIMIT = 64.f, GROWTH_STOP = 16.f;

// Whether A is certainly not singular, without a factorisation, so that none is needed for the report of a singular one: with its columns
// divided by their diagonal entries it is a matrix of signs and X, ||X||_2 < 1, seen from the Frobenius norm of X, or, which is less by up
// to the fourth root of d, from that of X^T X (one product, at d = 128, where the layer's A = I + 0.1 N / sqrt(d) needs it).  False also for
// anything that vanishes, overflows or is not finite on the way.
template <int D>
__device__ __forceinline__ bool certainly_regular(Pair<D>& W, float* s_part, Cols<D>& A, int w, int lane, int i, int g) {
  using C = Cfg<D>;
  float on[C::RB];
  diagonal_sizes<D>(A, on, w, i, g);
  float sq = 0.f;
#pragma unroll
  for (int k = 0; k < C::RB; ++k) {
    on[k] = __builtin_amdgcn_rcpf(on[k]);
    sq = __builtin_fmaf(0.f, on[k], sq);  // (not a number for a diagonal entry of 0)
  }
#pragma unroll
  for (int r = 0; r < C::NT; ++r)
#pragma unroll
    for (int k = 0; k < C::RB; ++k)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float x = r == C::RB * w + k && 4 * g + v == i ? 0.f : A[r][k][v] * on[k];
        if constexpr (D == 128) A[r][k][v] = x;
        else sq = __builtin_fmaf(x, x, sq);
      }
  if constexpr (D == 128) {
    SplitCols<D, C::RB> t;
    split_cols<D, C::RB>(A, t);
    store_split_T<D>(W, 0, t, w, i, g);
    lds_barrier();
    gemm_split<D, C::RB>(A, W, 0, t, i, g);
#pragma unroll
    for (int r = 0; r < C::NT; ++r)
#pragma unroll
      for (int k = 0; k < C::RB; ++k)
#pragma unroll
        for (int v = 0; v < 4; ++v) sq = __builtin_fmaf(A[r][k][v], A[r][k][v], sq);
  }
  sq = sum64(sq);
  if (lane == 0) s_part[w] = sq;
  lds_barrier();
  float all = 0.f;
#pragma unroll
  for (int ww = 0; ww < C::NW; ++ww) all += s_part[ww];
  return uniform(all < 0.9f ? 1 : 0) != 0;
}

// One round of the units below: a lane's s, and all of them in the notes (the last round's and the new ones side by side).  One barrier,
// the units are to be read behind another one.
template <int D>
__device__ __forceinline__ void next_state_units(Pair<D>& W, const Cols<D>& A, float (&s)[Cfg<D>::RB], int w, int i, int g) {
  using C = Cfg<D>;
  float* const units = state_units<D>(W);
#pragma unroll
  for (int k = 0; k < C::RB; ++k) {
    float big = 0.f;
#pragma unroll
    for (int r = 0; r < C::NT; ++r) {
      const floatx4 y = *reinterpret_cast<const floatx4*>(units + 16 * r + 4 * g);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float x = (r == C::RB * w + k && 4 * g + v == i) ? 0.f : __builtin_fabsf(A[r][k][v]) * y[v];
        big = __builtin_fmaxf(big, x);
      }
    }
    big = column_max(big);
    s[k] = big == 0.f ? s[k] : __builtin_fmaxf(s[k], unit_above(big));
    column_units<D>(W)[16 * (C::RB * w + k) + i] = s[k];
  }
  lds_barrier();
#pragma unroll
  for (int k = 0; k < C::RB; ++k) units[16 * (C::RB * w + k) + i] = s[k];
}
// Units of the states and controls of a problem, powers of two in the notes behind the pair: for state k just above the largest of
// sqrt(Q_kk), sqrt(Q_T,kk) and |A_ik| times that of state i, what it costs by itself and through the states it moves in one step; for
// control k just above sqrt(R_kk).  Written x' = D x, u' = V u, a problem's matrices do not depend on the units it came in and no entry of
// A or H is much larger than 1; split operands need that, as they keep 40 binary digits below the largest entry of a wavefront's
// columns.  A state without a cost of its own takes that of the states it reaches, round after round; one that reaches none has no
// influence on the others and counts for next to nothing.  Returns whether the units are used; within a factor of 16 they are all 1 and
// the digits that split operands have beyond float32 do (from 32 on what squaring itself loses shows too: a power's largest entries are
// then those that the units make large; bfloat16 inputs, T = 16, P_0 1e-5 for 9e-7).  The judgement costs 2 % of a call (d = 64, T = 16,
// 8192 problems 1.39 -> 1.41 ms); in functions of their own the scalings cost 15 % of every call, by the registers that the paths share,
// and at d = 128 in float32 they cost less without branches around them (T = 16, 2048 problems 2.51 -> 2.63 ms for 2.74, bfloat16 2.57 ->
// 2.70 for 2.75).
template <int D, typename TIn>
__device__ __forceinline__ bool publish_problem_units(Pair<D>& W, const Cols<D>& A, const TIn* Qp, const TIn* QTp, const TIn* Rp,
                                                      int w, int i, int g) {
  using C = Cfg<D>;
  float* const units = state_units<D>(W);
  float s[C::RB];
#pragma unroll
  for (int k = 0; k < C::RB; ++k) {
    const int j = 16 * (C::RB * w + k) + i;
    const long on = (long)j * (D + 1);
    const auto q = read1(Qp, on), qt = read1(QTp, on), r = read1(Rp, on);
    const float cost = __builtin_fmaxf(__builtin_fabsf(widen(q)), __builtin_fabsf(widen(qt)));
    s[k] = cost == 0.f ? 0.f : unit_of_square(cost);
    units[j] = s[k];
    control_units<D>(W)[j] = unit_of_square(__builtin_fabsf(widen(r)));
  }
  lds_barrier();
  next_state_units<D>(W, A, s, w, i, g);
  const bool controls = spread_above<D, 4>(control_units<D>(W), g), states = spread_above<D, 4>(column_units<D>(W), g);
  float lo = 1.f;  // the smallest unit
  if (__builtin_expect(states, 0)) {  // (also where a state has none yet)
    int open = D + 1, before;
    do {
      before = open;
      open = 0;
      lo = __builtin_inff();
      for (int r = 0; r < C::NT; ++r) {
        const floatx4 y = *reinterpret_cast<const floatx4*>(column_units<D>(W) + 16 * r + 4 * g);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          lo = y[v] != 0.f && y[v] < lo ? y[v] : lo;
          open += __popcll(__ballot(y[v] == 0.f));
        }
      }
      open = uniform(open);
      lds_barrier();
      if (open != 0 && open < before) {
        next_state_units<D>(W, A, s, w, i, g);
        lds_barrier();
      }
    } while (open != 0 && open < before);
    lo = column_max(lo < __builtin_inff() ? power_inverse(lo) : 0.f);
    lo = lo == 0.f ? 1.f : power_inverse(lo);  // (no costs at all)
  }
  lds_barrier();
#pragma unroll
  for (int k = 0; k < C::RB; ++k) {
    const int j = 16 * (C::RB * w + k) + i;
    units[j] = !states ? 1.f : s[k] == 0.f ? __builtin_fmaxf(lo * 0x1p-40f, 0x1p-80f) : s[k];
    control_units<D>(W)[j] = controls ? control_units<D>(W)[j] : 1.f;
  }
  lds_barrier();
  return states || controls;
}
// m <- diag(u) m diag(1 / v), u and v in LDS: a map in units of its own
template <int D>
__device__ __forceinline__ void map_in_units(Cols<D>& m, const float* u, const float* v, int w, int i, int g) {
  float x[Cfg<D>::RB];
#pragma unroll
  for (int k = 0; k < Cfg<D>::RB; ++k) x[k] = power_inverse(v[16 * (Cfg<D>::RB * w + k) + i]);
  scale_rows<D>(m, u, g);
  scale_columns<D>(m, x);
}
// the same of its transpose, m = M^T, and back from units: diag(1 / v) m diag(u)
template <int D>
__device__ __forceinline__ void map_in_units_T(Cols<D>& m, const float* u, const float* v, int w, int i, int g) {
  float x[Cfg<D>::RB];
#pragma unroll
  for (int k = 0; k < Cfg<D>::RB; ++k) x[k] = u[16 * (Cfg<D>::RB * w + k) + i];
  scale_rows<D, true>(m, v, g);
  scale_columns<D>(m, x);
}
// diag(1 / u) m diag(1 / u): a cost
template <int D>
__device__ __forceinline__ void cost_in_units(Cols<D>& m, const float* u, int w, int i, int g) {
  float x[Cfg<D>::RB];
#pragma unroll
  for (int k = 0; k < Cfg<D>::RB; ++k) x[k] = power_inverse(u[16 * (Cfg<D>::RB * w + k) + i]);
  scale_rows<D, true>(m, u, g);
  scale_columns<D>(m, x);
}

// One column tile per wavefront at d >= 64 (build.py): two at d = 128 leave one wavefront a SIMD (T = 16, 8192 problems 14.9 against
// 11.6 ms), at d = 64 two wavefronts (T = 8, 16384 problems 2.73 against 2.55 ms with one tile and three wavefronts).  The registers
// do not hold all of it (float32 / bfloat16 inputs 100 / 114 spilled at d = 64, 444 / 516 at d = 128, around the inverse), which costs less
// than another wavefront would.
// The recursion and the solves of the problems given up are in a kernel of their own: inlined here they spilled many more.
// Measured, products in float32 with row blocks in registers -> split products -> this, with A proved regular instead of factored, the
// inverse by blocks and the chain's priority (and at d = 128 the operands' largest entry by the IEEE maximum), ms: d = 64, T = 8, 16384
// problems 3.21 -> 2.40 -> 2.27, T = 64, 4099 problems 1.50 -> 0.944 -> 0.905; d = 128, T = 16, 8192 problems 16.3 -> 10.3 -> 9.63;
// bfloat16 inputs, T = 32, 4096 problems 9.77 -> 6.25 -> 5.72.  Errors against float64 with products in float32 -> split: 0.87e-6 ->
// 0.65e-6, 0.77e-6 -> 0.56e-6, 1.9e-6 -> 1.3e-6, 2.4e-6 -> 1.5e-6; no larger since.
template <int D, typename TIn>
__global__ void __launch_bounds__(Cfg<D>::NTHR, (D) == 64 ? 3 : 2) squaring_kernel(const DoublingArgs da) {
  using C = Cfg<D>;
  using Split = SplitCols<D, C::RB>;
  constexpr int L = 0, R = 1;  // the halves of the pair
  constexpr bool PARK = D == 128;  // the transpose of A_e waits in LDS while an inverse is formed
  __shared__ __attribute__((aligned(16))) float W[C::PAIR];
  __shared__ __attribute__((aligned(16))) SolveScratch<D> S;
  __shared__ float s_red[C::NW];
  __shared__ float s_max[C::NW];  // per wavefront: max |I + G H| of the matrix being inverted
  const SolveArgs& p = da.s;
  float* const WL = W;
  float* const WR = W + D;
  float* const wsP = p.ws + (long)blockIdx.x * D * D;  // P, as the registers hold it

  for (long long prob = blockIdx.x; prob < p.n; prob += gridDim.x) {
    const int tid = threadIdx.x + opaque_zero(), lane = tid & 63, w = uniform(tid >> 6), i = lane & 15, g = lane >> 4;
    const TIn* Ap = reinterpret_cast<const TIn*>(p.A) + prob * p.sA;
    const TIn* Bp = reinterpret_cast<const TIn*>(p.B) + prob * p.sB;
    const TIn* Qp = reinterpret_cast<const TIn*>(p.Q) + prob * p.sQ;
    const TIn* Rp = reinterpret_cast<const TIn*>(p.R) + prob * p.sR;
    const TIn* x0p = reinterpret_cast<const TIn*>(p.x0) + prob * p.sx0;
    const TIn* QTp = da.p_from_qt ? reinterpret_cast<const TIn*>(p.QT) + prob * p.sQT : Qp;
    uint32_t give_up = 0;   // whom the problem is handed to
    bool pivoted = false;   // the inverses search pivots, from the first large mu on

    // (the word's writer is the thread that writes the first of u_0 in emit_gain)
    auto hand_over = [&](uint32_t how) {
      if (threadIdx.x == 0) reinterpret_cast<uint32_t*>(p.u0)[prob * D] = how;
      __syncthreads();  // every wavefront has left the pair
    };

    Split a, at;  // A_e and its transpose
    Cols<D> G, H;
    bool own;  // whether the problem is written in units of its own
    constexpr bool ALWAYS = D == 128 && sizeof(TIn) == 4;  // (multiplied by them in any case, which is exact)
    const float* const xu = state_units<D>(W);
    const float* const uu = control_units<D>(W);
    {
      Cols<D> m;
      load_cols<D, TIn>(Ap, m, w, i, g);
      own = publish_problem_units<D, TIn>(W, m, Qp, QTp, Rp, w, i, g);
      if (ALWAYS || __builtin_expect(own, 0)) map_in_units<D>(m, xu, xu, w, i, g);
      split_cols<D, C::RB>(m, a);
    }
    // ---- set-up: G = B R^{-1} B^T, H = Q; P = Q_T when it is a matrix of its own
    const int thread = tid;
    {
      // (formed anew at d = 128, or its address arithmetic pushes the element into memory: T = 16, 8192 problems 10.64 -> 9.61 ms)
      const int tid = D == 128 ? (int)threadIdx.x + opaque_zero() : thread;
      const int lane = tid & 63, w = uniform(tid >> 6), i = lane & 15, g = lane >> 4;
      Cols<D> r, bt;
      Split t;
      load_cols_T<D, TIn>(Bp, bt, w, i, g);
      zero_cols<D>(r);
      add_sym_cols<D, TIn>(Rp, r, w, i, g);
      if (ALWAYS || __builtin_expect(own, 0)) {
        cost_in_units<D>(r, uu, w, i, g);
        map_in_units_T<D>(bt, xu, uu, w, i, g);
      }
      split_cols<D, C::RB>(bt, t);
      store_split_T<D>(W, L, t, w, i, g);  // B
      if (invert_or_solve<D>(W, r, bt, t, w, lane, i, g)) {  // R^{-1} B^T, or R is not positive definite
        hand_over(HANDED_TO_PRODUCT);
        continue;
      }
      split_cols<D, C::RB>(bt, t);
      gemm_split<D, C::RB>(G, W, L, t, i, g);
      lds_barrier();
      // G is symmetric up to rounding; make it exactly so
      store_cols_T<D>(WR, G, w, i, g);
      load_cols_T<D, TIn>(Ap, bt, w, i, g);
      if (ALWAYS || __builtin_expect(own, 0)) map_in_units_T<D>(bt, xu, xu, w, i, g);
      split_cols<D, C::RB>(bt, at);
      zero_cols<D>(H);
      add_sym_cols<D, TIn>(Qp, H, w, i, g);
      if (ALWAYS || __builtin_expect(own, 0)) cost_in_units<D>(H, xu, w, i, g);
      lds_barrier();
      read_cols<D>(WR, r, w, i, g);
#pragma unroll
      for (int x = 0; x < C::NT; ++x)
#pragma unroll
        for (int k = 0; k < C::RB; ++k) G[x][k] = 0.5f * (G[x][k] + r[x][k]);
    }
    bool have_p = da.p_from_qt != 0, at_QT = have_p;  // at_QT: P is still Q_T
    if (have_p) {
      Cols<D> t;
      zero_cols<D>(t);
      add_sym_cols<D, TIn>(QTp, t, w, i, g);
      if (ALWAYS || __builtin_expect(own, 0)) cost_in_units<D>(t, xu, w, i, g);
      keep_cols<D>(wsP, t, tid);
    }
    lds_barrier();

    // ---- P_1 by binary powering of the one-step map (see ttc_doubling.hpp).  A turn of the loop either applies e to P or squares
    // it: both begin with the inverse of a matrix I + (symmetric)(symmetric), formed transposed, so that its columns are the rows
    // of the inverse wanted as a left operand.
    bool p_is_H = false;   // P_1 = H_e: the last bit met no P
    bool bit_done = false; // P has had the current bit of m
    float mu_prev = 0.f;   // max |I + G_e H_e| of the squaring before, 0 before the first
    bool stay = false;     // e is not squared any further, but applied once for each factor of it that is left
    for (int m = da.m; m;) {
      const int tid = threadIdx.x + opaque_zero(), lane = tid & 63, w = uniform(tid >> 6), i = lane & 15, g = lane >> 4;
      bool apply = false;
      if (!bit_done && ((m & 1) || stay)) {
        apply = have_p;
        if (!have_p) {  // f_e(0) = H_e
          have_p = true;
          if (m == 1) {  // and e is not touched again
            p_is_H = true;
            break;
          }
          keep_cols<D>(wsP, H, tid);
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
      Cols<D> s;
      {
        Split l, r;
        if (apply) {
          zero_cols<D>(s);
          add_kept_cols<D>(wsP, s, tid);
          split_cols<D, C::RB>(s, r);
          split_cols<D, C::RB>(G, l);
        } else {
          split_cols<D, C::RB>(H, l);
          split_cols<D, C::RB>(G, r);
        }
        store_split_T<D>(W, L, l, w, i, g);
        eye_cols<D>(s, w, i, g);
        lds_barrier();
        gemm_split<D, C::RB, true>(s, W, L, r, i, g);  // (I + P G)^T, or (I + G H)^T
      }
      {
        float big = 0.f;
#pragma unroll
        for (int r = 0; r < C::NT; ++r)
#pragma unroll
          for (int k = 0; k < C::RB; ++k)
#pragma unroll
            for (int v = 0; v < 4; ++v) {  // as bits: NaN on top
              const float x = __builtin_fabsf(s[r][k][v]);
              big = __float_as_uint(x) > __float_as_uint(big) ? x : big;
            }
        big = wave_max_nonneg(big);
        if (lane == 0) s_max[w] = big;
      }
      lds_barrier();
      uint32_t mu_bits = 0;
#pragma unroll
      for (int ww = 0; ww < C::NW; ++ww) {
        const uint32_t b = __float_as_uint(s_max[ww]);
        mu_bits = b > mu_bits ? b : mu_bits;
      }
      const float mu = __uint_as_float(uniform(mu_bits));
      const bool only_H = !apply && m == 1 && !have_p;  // the last squaring, and P is still 0: A and G of the square are not needed
      if (!(mu <= (apply ? (at_QT ? da.qt_limit : LATE_LIMIT) : mu_prev == 0.f ? p.growth_limit : LATE_LIMIT))) {
        give_up = HANDED_TO_RECURSION;
        break;
      }
      if (apply) {
        at_QT = false;
      } else {
        // growth of an unstable open loop: mu - 1 has grown by r, and the square of e will make it grow by r^2 at least
        const float up = mu - 1.f, up_prev = mu_prev - 1.f;
        if (!only_H && mu_prev != 0.f && up > 1.f && up > 2.f * up_prev && up * up * up > GROWTH_STOP * up_prev * up_prev) {
          stay = true;
          m *= 2;
          lds_barrier();  // s_max is written again at once
          continue;
        }
        mu_prev = mu;
      }
      pivoted = pivoted || mu > IN_ORDER_MAX;
      // The transpose of A_e, the operand that the products behind the inverse need last, waits in LDS as the left operand A_e:
      // 32 registers at d = 128, where what does not fit goes to memory (16 of its 16-byte pieces a lane cost as much as three products).
      if constexpr (PARK) store_split_T<D>(W, L, at, w, i, g);
      int flag;
      if (__builtin_expect(!pivoted, 1)) {
        flag = invert_cols<D>(WR, s, w, lane, PIVOT_MIN);
      } else {
        if constexpr (PARK) {
          read_split<D>(W, L, at, w, i, g);
          lds_barrier();
        }
        store_cols<D>(WL, C::PITCH, s, w, i, g);
        set_half_identity<D>(WR, tid);
        __syncthreads();
        flag = lds_solve_aside<D>(W, S, tid);
        read_cols<D>(WR, s, w, i, g);
        lds_barrier();
        if constexpr (PARK) store_split_T<D>(W, L, at, w, i, g);
      }
      if (flag) {  // a pivot below PIVOT_MIN, or none at all
        give_up = HANDED_TO_PRODUCT;
        break;
      }
      Split t;
      split_cols<D, C::RB>(s, t);
      store_split_T<D>(W, R, t, w, i, g);  // M = (I + P G)^{-1}, or (I + G H)^{-1}
      if (__builtin_expect(apply, 0)) {
        if constexpr (PARK) read_split<D>(W, L, at, w, i, g);
        zero_cols<D>(s);
        add_kept_cols<D>(wsP, s, tid);
        split_cols<D, C::RB>(s, t);
        store_split_T<D>(W, L, t, w, i, g);  // P (the rows just read are this wavefront's own)
        lds_barrier();
        gemm_split<D, C::RB>(s, W, L, a, i, g);  // P A
        split_cols<D, C::RB>(s, t);
        gemm_split<D, C::RB>(s, W, R, t, i, g);  // V = M P A
        split_cols<D, C::RB>(s, t);
        lds_barrier();
        store_split_T<D>(W, L, a, w, i, g);  // A^T
        lds_barrier();
#pragma unroll
        for (int r = 0; r < C::NT; ++r)
#pragma unroll
          for (int k = 0; k < C::RB; ++k) s[r][k] = H[r][k];
        gemm_split<D, C::RB, true>(s, W, L, t, i, g);  // P <- H_e + A_e^T (I + P G_e)^{-1} P A_e
        keep_cols<D>(wsP, s, tid);
        lds_barrier();
        if (stay) --m;
        else bit_done = true;
        continue;
      }
      // e <- e o e
      bit_done = false;
      Split ma;
      if (only_H) {
        split_cols<D, C::RB>(H, t);
        store_split_T<D>(W, L, t, w, i, g);  // H
        lds_barrier();
        gemm_split<D, C::RB>(s, W, R, a, i, g);  // M A
        split_cols<D, C::RB>(s, ma);
        gemm_split<D, C::RB>(s, W, L, ma, i, g);  // V = H M A
        split_cols<D, C::RB>(s, t);
        lds_barrier();
        store_split_T<D>(W, R, a, w, i, g);  // A^T
        lds_barrier();
        gemm_split<D, C::RB, true>(H, W, R, t, i, g);  // H' = H + A^T V
        lds_barrier();
      } else {
        if constexpr (!PARK) store_split_T<D>(W, L, at, w, i, g);  // A
        lds_barrier();
        gemm_split<D, C::RB>(s, W, R, a, i, g);  // M A
        split_cols<D, C::RB>(s, ma);
        split_cols<D, C::RB>(G, t);
        gemm_split<D, C::RB>(s, W, R, t, i, g);  // M G, symmetric
        split_cols<D, C::RB>(s, t);
        lds_barrier();
        store_split_T<D>(W, R, t, w, i, g);
        if constexpr (PARK) read_split<D>(W, L, at, w, i, g);
        lds_barrier();
        gemm_split<D, C::RB>(s, W, R, at, i, g);  // M G A^T
        split_cols<D, C::RB>(s, t);
        gemm_split<D, C::RB, true>(G, W, L, t, i, g);  // G' = G + A M G A^T
        gemm_split<D, C::RB>(s, W, L, ma, i, g);       // A' = A M A
        split_cols<D, C::RB>(H, t);
        lds_barrier();
        store_split_T<D>(W, L, t, w, i, g);  // H
        store_split_T<D>(W, R, a, w, i, g);  // A^T
        split_cols<D, C::RB>(s, a);
        lds_barrier();
        {
          Cols<D> v;
          gemm_split<D, C::RB>(v, W, L, ma, i, g);  // V = H M A
          split_cols<D, C::RB>(v, t);
        }
        gemm_split<D, C::RB, true>(H, W, R, t, i, g);  // H' = H + A^T V
        lds_barrier();
        store_cols<D>(WL, C::PITCH, s, w, i, g);
        lds_barrier();
        read_cols_T<D>(WL, s, w, i, g);
        split_cols<D, C::RB>(s, at);
        lds_barrier();
      }
    }

    // ---- last step, with the problem's own matrices: as printed
    if (!give_up) {
      const int tid = threadIdx.x + opaque_zero(), lane = tid & 63, w = uniform(tid >> 6), i = lane & 15, g = lane >> 4;
      if (!p_is_H) {
        zero_cols<D>(H);
        add_kept_cols<D>(wsP, H, tid);
      }
      store_cols_T<D>(WR, H, w, i, g);
      __syncthreads();
      symmetrise_half<D>(WR, tid);
      __syncthreads();
      Cols<D> wk, pn, b, r, t;
      float e[C::RB];
      step_operands<D, TIn>(
          W, Ap, Bp, [&](Cols<D>& m, int w, int i, int g) { add_sym_cols<D, TIn>(Rp, m, w, i, g); }, pn, b, r, t, e, w, i, g);
      if (ALWAYS || __builtin_expect(own, 0)) {
        map_in_units<D>(t, xu, xu, w, i, g);  // (A - E: what is on the diagonal stays)
        map_in_units<D>(b, xu, uu, w, i, g);
        cost_in_units<D>(r, uu, w, i, g);
      }
      if (__builtin_expect(step_needs_units<D>(W, pn, b, t, e, w, i, g), 0)) {  // others than the problem's
        give_up = HANDED_TO_RECURSION;
      } else if (step_products<D>(W, pn, b, r, t, e, wk, w, lane, i, g)) {
        give_up = HANDED_TO_PRODUCT;
      } else {
        if (ALWAYS || __builtin_expect(own, 0)) {  // back to the units the problem came in
          float x[C::RB];
#pragma unroll
          for (int k = 0; k < C::RB; ++k) x[k] = xu[16 * (C::RB * w + k) + i];
          scale_rows<D>(pn, xu, g);
          scale_columns<D>(pn, x);
          map_in_units_T<D>(wk, xu, uu, w, i, g);
        }
        emit_step<D, TIn>(W, s_red, p, prob, wk, pn, Qp, x0p, 0, tid);
      }
    }
    // ---- a singular A is reported, although nothing here divides by A: by the sequential product.  Here, where no register of the problem's
    // is in use any more (ahead of the set-up, inverses got slower by more than the factorisation that this leaves out).
    if (give_up != HANDED_TO_PRODUCT) {
      __syncthreads();  // every wavefront has left the pair and s_max
      const int tid = threadIdx.x + opaque_zero(), lane = tid & 63, w = uniform(tid >> 6), i = lane & 15, g = lane >> 4;
      Cols<D> m;
      load_cols<D, TIn>(Ap, m, w, i, g);
      if (__builtin_expect(!certainly_regular<D>(W, s_max, m, w, lane, i, g), 0)) {
        lds_barrier();
        floatx4 none[C::NT][1];  // no right-hand sides
        load_cols<D, TIn>(Ap, m, w, i, g);
        if (__builtin_expect(solve_cols<D, 0>(WR, m, none, w, lane, PIVOT_MIN_A), 0)) {
          load_half<D, TIn, false>(WL, Ap, tid);
          __syncthreads();
          if (lds_factor_aside<D>(W, S, tid)) give_up = HANDED_TO_PRODUCT;
        }
      }
      __syncthreads();
    }
    if (give_up) hand_over(give_up);
  }
}

}  // namespace ttc
