// Time-heterogeneous problems: A_t, B_t, Q_t, R_t vary over the horizon (the general statement of
// Prop. 3.1; the paper's "time-heterogeneous parameterization", Sec. 4).
//
// With every factor Sigma_t of Thm 3.3 different, nothing can be prepared once per problem: each factor
// would need its own A_t^{-1} and G_t = B_t R_t^{-1} B_t^T, two dense solves before the factor is even
// applied, and a re-base on top.  Re-basing after every factor turns the iteration into the backward
// recursion of Prop. 3.1 itself, and its printed form needs one solve per step, with a positive
// definite matrix (no pivot search):
//     S_s = R_s + B_s^T P_{s+1} B_s,   W_s = S_s^{-1} B_s^T P_{s+1} A_s,   K_s = -W_s        (Eq. "decode")
//     P_s = Q[s-1] + A_s^T P_{s+1} A_s - (B_s^T P_{s+1} A_s)^T W_s   (P_T = Q[T-1], no Q on x_0)  (Eq. "riccati")
// Six products and one dense solve per step; the value matrix stays on chip for the whole horizon, the
// step's matrices are streamed from HBM once each.
#pragma once
#include "ttc_common.hpp"
#include "ttc_small.hpp"
#include "ttc_columns.hpp"
#include "ttc_rollout.hpp"

namespace ttc {


// accumulator rows of this wavefront <- row-major global matrix of input element type
template <int D, typename TIn>
__device__ __forceinline__ void load_rows_input(const TIn* src, floatx4 (&acc)[Cfg<D>::RB][Cfg<D>::NT], int w, int i, int g) {
  using C = Cfg<D>;
#pragma unroll
  for (int rb = 0; rb < C::RB; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int h = 0; h < C::NH; ++h) {
        const long off = (long)(16 * (C::RB * w + rb) + 4 * g + v) * D + 16 * C::VEC * h + C::VEC * i;
        if constexpr (C::VEC == 4) {
          const floatx4 t = ld4<TIn>(src, off);
#pragma unroll
          for (int tp = 0; tp < 4; ++tp) acc[rb][h * 4 + tp][v] = t[tp];
        } else {
#pragma unroll
          for (int tp = 0; tp < C::VEC; ++tp) acc[rb][h * C::VEC + tp][v] = ld1<TIn>(src, off + tp);
        }
      }
}

// The outputs from the last step taken, as riccati_step leaves it: wk = -K_0 and pn = P_0 (no cost on x_0).
template <int D, typename TIn>
__device__ __forceinline__ void emit_step(float* W, float* s_red, const SolveArgs& p, long long prob, const Cols<D>& wk,
                                          const Cols<D>& pn, const TIn* Qflag, const TIn* x0p, int info, int tid) {
  using C = Cfg<D>;
  const int lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
  float* const WL = W;
  float* const WR = W + D;
  __syncthreads();  // every wavefront has left the pair
  store_cols_T<D>(WL, pn, w, i, g);
  store_cols<D>(WR, C::PITCH, wk, w, i, g);
  __syncthreads();
  symmetrise_half<D>(WL, tid);
  __syncthreads();
  floatx4 acc[C::RB][C::NT];
  load_rows<D>(WR, acc, w, i, g);  // rows of -K_0
  emit_gain<D, TIn>(p, prob, acc, x0p, info, tid);
  emit_value<D, TIn>(p, prob, WL, Qflag, x0p, info, s_red, tid);
}

// The whole backward recursion of one problem by one workgroup, from P_T to the outputs P_0, K_0, u_0, value and
// info: T calls of riccati_step.  Step s reads A, B, R at As + s*tA, Bs + s*tB, Rs + s*tR and the stage cost on
// the state it starts from at Qs + (s-1)*tQ (none for s = 0); zero strides give the time-invariant problem.
// The terminal value matrix is PTf (float32) if given, else PT (input element type).  info_base is added to the
// index (1 = the step taken first, s = T-1) of the step whose solve broke down; the result is what info becomes.  All
// threads must call it.
template <int D, typename TIn>
__device__ __forceinline__ int riccati_problem(Pair<D>& W, float* s_red, const SolveArgs& p,
                                                long long prob, int T, const TIn* As, const TIn* Bs, const TIn* Qs,
                                                const TIn* Rs, long long tA, long long tB, long long tQ, long long tR,
                                                const TIn* PT, const float* PTf, const TIn* Qflag, const TIn* x0p,
                                                int info_base, int tid) {
  float* const WR = W + D;
  int info = 0;
  if (PTf) load_half<D, float, false>(WR, PTf, tid);
  else load_half<D, TIn, false>(WR, PT, tid);
  __syncthreads();
  symmetrise_half<D>(WR, tid);
  __syncthreads();
  for (int s = T - 1; s >= 0; --s) {
    Cols<D> wk, pn;
    const int flag = riccati_step<D, TIn>(W, As + (long long)s * tA, Bs + (long long)s * tB, Rs + (long long)s * tR, wk,
                                          pn, tid);
    if (flag && !info) info = info_base + T - s;
    if (s >= 1 && !info) {
      next_value_matrix<D, TIn>(W, Qs + (long long)(s - 1) * tQ, pn, tid + opaque_zero());
    } else {
      emit_step<D, TIn>(W, s_red, p, prob, wk, pn, Qflag, x0p, info, tid);
      break;
    }
  }
  return info;
}

template <int D, typename TIn>
__global__ void __launch_bounds__(Cfg<D>::NTHR, TTC_COLS_WAVES(D)) solve_tv_kernel(const TvArgs ta) {
  using C = Cfg<D>;
  __shared__ __attribute__((aligned(16))) float W[C::PAIR];
  __shared__ float s_red[C::NW];
  const SolveArgs& p = ta.s;

  for (long long prob = blockIdx.x; prob < p.n; prob += gridDim.x) {
    const int tid = threadIdx.x + opaque_zero();
    const TIn* Ap = reinterpret_cast<const TIn*>(p.A) + prob * p.sA;
    const TIn* Bp = reinterpret_cast<const TIn*>(p.B) + prob * p.sB;
    const TIn* Qp = reinterpret_cast<const TIn*>(p.Q) + prob * p.sQ;
    const TIn* Rp = reinterpret_cast<const TIn*>(p.R) + prob * p.sR;
    const TIn* x0p = reinterpret_cast<const TIn*>(p.x0) + prob * p.sx0;
    riccati_problem<D, TIn>(W, s_red, p, prob, p.T, Ap, Bp, Qp, Rp, ta.tA, ta.tB, ta.tQ, ta.tR,
                            Qp + (long long)(p.T - 1) * ta.tQ, ta.PT ? ta.PT + prob * ta.sPT : nullptr, Qp, x0p, 0, tid);
  }
}

// Roll-out of a time-heterogeneous problem (Alg. 1 with r = 0): the backward sweep of solve_tv_kernel
// keeping every gain K_s in the workspace, then the closed-loop forward sweep
// u_s = K_s x_s, x_{s+1} = A_s x_s + B_s u_s with the cost sum_s u_s^T R_s u_s + x_{s+1}^T Q[s] x_{s+1}.
template <int D, typename TIn>
__global__ void __launch_bounds__(Cfg<D>::NTHR, TTC_COLS_WAVES(D)) rollout_tv_kernel(const TvRolloutArgs ta) {
  using C = Cfg<D>;
  __shared__ __attribute__((aligned(16))) float W[C::PAIR];
  __shared__ float s_red[C::NW];
  __shared__ __attribute__((aligned(16))) float s_x[D], s_u[D], s_xn[D];
  const RolloutArgs& p = ta.r;
  float* const WR = W + D;
  float* const wsK = p.ws + (long)blockIdx.x * p.T * D * D;  // K_0 .. K_{T-1}, row-major

  for (long long prob = blockIdx.x; prob < p.n; prob += gridDim.x) {
    const TIn* Ap = reinterpret_cast<const TIn*>(p.A) + prob * p.sA;
    const TIn* Bp = reinterpret_cast<const TIn*>(p.B) + prob * p.sB;
    const TIn* Qp = reinterpret_cast<const TIn*>(p.Q) + prob * p.sQ;
    const TIn* Rp = reinterpret_cast<const TIn*>(p.R) + prob * p.sR;
    const TIn* x0p = reinterpret_cast<const TIn*>(p.x0) + prob * p.sx0;
    int info = 0;
    {
      const int tid = threadIdx.x + opaque_zero(), lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
      load_half<D, TIn, false>(WR, Qp + (long long)(p.T - 1) * ta.tQ, tid);  // P_T = Q_T
      __syncthreads();
      symmetrise_half<D>(WR, tid);
      __syncthreads();
      // ---- backward sweep
      for (int s = p.T - 1; s >= 0; --s) {
        Cols<D> wk, pn;
        const int flag = riccati_step<D, TIn>(W, Ap + (long long)s * ta.tA, Bp + (long long)s * ta.tB,
                                              Rp + (long long)s * ta.tR, wk, pn, tid);
        if (flag && !info) info = p.T - s;
        store_cols<D, -1>(wsK + (long)s * D * D, D, wk, w, i, g);  // K_s
        if (s >= 1) next_value_matrix<D, TIn>(W, Qp + (long long)(s - 1) * ta.tQ, pn, tid);
      }
    }
    __syncthreads();  // gains visible to the whole workgroup

    // ---- forward sweep
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int r = tid / (C::NTHR / D), part = tid % (C::NTHR / D);
    if (tid < D) s_x[tid] = ld1<TIn>(x0p, tid);
    __syncthreads();
    float cpart = 0.f;
    if (p.X && tid < D) p.X[prob * (long)(p.T + 1) * D + tid] = s_x[tid];
    for (int t = 0; t < p.T; ++t) {
      RowShare<D> Kr;  // the step's five reads side by side
      RowShareOf<D, TIn> Ar, Br, Rr, Qr;
      Kr.load(rows_of<D, float>(wsK + (long)t * D * D), tid);
      Ar.load(rows_of<D, TIn>(Ap + (long long)t * ta.tA), tid);
      Br.load(rows_of<D, TIn>(Bp + (long long)t * ta.tB), tid);
      Rr.load(rows_of<D, TIn>(Rp + (long long)t * ta.tR), tid);
      Qr.load(rows_of<D, TIn>(Qp + (long long)t * ta.tQ), tid);
      TTC_SCHED_BARRIER();
      const float u = Kr.dot(s_x, tid);
      const float ax = Ar.dot(s_x, tid);
      if (part == 0) s_u[r] = u;
      lds_barrier();
      const float ru = Rr.dot(s_u, tid);
      const float xn = ax + Br.dot(s_u, tid);
      if (part == 0) {
        cpart += u * ru;
        s_xn[r] = xn;
        p.U[(prob * p.T + t) * (long)D + r] = info ? __builtin_nanf("") : u;
        if (p.X) p.X[(prob * (p.T + 1) + t + 1) * (long)D + r] = info ? __builtin_nanf("") : xn;
      }
      lds_barrier();
      const float qx = Qr.dot(s_xn, tid);
      if (part == 0) {
        cpart += xn * qx;
        s_x[r] = xn;
      }
      lds_barrier();
    }
    cpart = sum64(cpart);
    if (lane == 0) s_red[w] = cpart;
    __syncthreads();
    if (tid == 0) {
      float cst = 0.f;
      for (int ww = 0; ww < C::NW; ++ww) cst += s_red[ww];
      if (p.cost) p.cost[prob] = info ? __builtin_nanf("") : cst;
      if (p.info) p.info[prob] = info;
    }
    __syncthreads();
  }
}

// The same at d = 16 with one or four problems per wavefront (see ttc_small.hpp).  At this size the accumulator layout of
// a matrix (lane (i, g) holds M[4g + v][i]) is at once its own B operand and the A operand of its transpose, so a step runs
// from register to register: P A, P B, then B^T (P B), B^T (P A), A^T (P A) straight from the loaded A, B; only S passes
// through LDS, on its way to a row per lane for the inverse.  Products of the wavefront's problems are interleaved.
// PPW = problems per wavefront: 4 for batches that fill the chip, 1 for small ones (the four rows of 16 lanes then all
// invert the same matrix; every per-problem loop runs once).

// accumulator layout of a row-major 16 x 16 matrix in memory, and of its transpose (a lane's four values are 16 bytes)
template <typename TIn>
__device__ __forceinline__ floatx4 load_acc16(const TIn* M, int i, int g) {
  floatx4 r;
#pragma unroll
  for (int v = 0; v < 4; ++v) r[v] = ld1<TIn>(M, (unsigned)(64 * g + i) + 16 * v);
  return r;
}
template <typename TIn>
__device__ __forceinline__ floatx4 load_accT16(const TIn* M, int i, int g) {
  return ld4<TIn>(M, (unsigned)(16 * i + 4 * g));
}

// acc[q] += L_q R_q for the wavefront's problems: a = the accumulator layout of L_q^T, b = that of R_q
template <int PPW>
__device__ __forceinline__ void mul16(floatx4 (&acc)[PPW], const floatx4 (&a)[PPW], const floatx4 (&b)[PPW]) {
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int q = 0; q < PPW; ++q) acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q][t], b[q][t], acc[q], 0, 0, 0);
}
template <int PPW>
__device__ __forceinline__ void zero16(floatx4 (&acc)[PPW]) {
#pragma unroll
  for (int q = 0; q < PPW; ++q) acc[q] = floatx4{0.f, 0.f, 0.f, 0.f};
}
// P <- (P + P^T) / 2, exactly symmetric: the transpose is formed on the matrix cores as P^T times the identity (exact)
template <int PPW>
__device__ __forceinline__ void symmetrise16(floatx4 (&P)[PPW], int i, int g) {
  floatx4 eye[PPW], t[PPW];
#pragma unroll
  for (int q = 0; q < PPW; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) eye[q][v] = (4 * g + v == i) ? 1.f : 0.f;
  zero16<PPW>(t);
  mul16<PPW>(t, P, eye);
#pragma unroll
  for (int q = 0; q < PPW; ++q) P[q] = 0.5f * (P[q] + t[q]);
}

// One backward step of Prop. 3.1 for the wavefront's problems.  On entry P holds P_{s+1} (symmetric), A, B the step's
// matrices and Rl(q) returns (the symmetric part of) R, asked for when it is needed; next() is called when A, B and R are
// no longer needed; on exit Wk = S^{-1} B^T P A = -K_s and
// pn = A^T P A - (B^T P A)^T Wk.  Wm: 16 x PITCH floats of LDS per problem.  Returns, per lane, a breakdown of the inverse.
// BLOCKS (one problem to a wavefront): the inverse by blocks of four pivots, the faster; without it by columns, every rounding as with four.
template <int PPW, bool BLOCKS = false, typename RLoad, typename Next>
__device__ __forceinline__ int riccati_step16(float (*Wm)[16 * Cfg<16>::PITCH], const floatx4 (&P)[PPW],
                                              const floatx4 (&A)[PPW], const floatx4 (&B)[PPW], RLoad&& Rl, Next&& next,
                                              floatx4 (&Wk)[PPW], floatx4 (&pn)[PPW], floatx4 (&S)[PPW],
                                              floatx4 (&Si)[PPW], int lane) {
  using C = Cfg<16>;
  const int i = lane & 15, g = lane >> 4;
  floatx4 PA[PPW], PB[PPW], F[PPW];
  zero16<PPW>(PB);
  mul16<PPW>(PB, P, B);  // P B
  zero16<PPW>(S);
  mul16<PPW>(S, B, PB);  // B^T P B
  zero16<PPW>(PA);
  mul16<PPW>(PA, P, A);  // P A
#pragma unroll
  for (int q = 0; q < PPW; ++q) S[q] += Rl(q);
  // the inverse (of S^T, that is of S up to rounding), its rows as the A operand
  int bad;
  if constexpr (PPW == 1) {
    zero16<PPW>(F);
    mul16<PPW>(F, B, PA);  // F = B^T P A
    zero16<PPW>(pn);
    mul16<PPW>(pn, A, PA);  // A^T P A
    next();
    Si[0] = S[0];
    bad = BLOCKS ? invert_spread16(Si[0], lane) : invert_columns16(Si[0], lane);
  } else {
#pragma unroll
    for (int q = 0; q < PPW; ++q) *reinterpret_cast<floatx4*>(Wm[q] + i * C::PITCH + 4 * g) = S[q];  // S^T, row-major
    wave_lds_sync();
    zero16<PPW>(F);
    mul16<PPW>(F, B, PA);
    zero16<PPW>(pn);
    mul16<PPW>(pn, A, PA);
    next();
    bad = invert_rows16(Wm[g & (PPW - 1)], lane);
#pragma unroll
    for (int q = 0; q < PPW; ++q) Si[q] = *reinterpret_cast<const floatx4*>(Wm[q] + i * C::PITCH + 4 * g);
  }
  zero16<PPW>(Wk);
  mul16<PPW>(Wk, Si, F);  // W = S^{-1} F
  // One step of refinement, W += S^{-1} (F - S W): an explicitly formed inverse leaves an error proportional to cond(S)
  // in W, which the cancellation in A^T P A - F^T W magnifies when control is cheap; the corrected W is as good as a
  // factor-and-solve.
  floatx4 res[PPW], neg[PPW];
#pragma unroll
  for (int q = 0; q < PPW; ++q) {
    res[q] = F[q];
    neg[q] = -S[q];  // the A operand of -S^T, the matrix that was inverted
  }
  mul16<PPW>(res, neg, Wk);
  mul16<PPW>(Wk, Si, res);
#pragma unroll
  for (int q = 0; q < PPW; ++q) neg[q] = -F[q];
  mul16<PPW>(pn, neg, Wk);  // - F^T W
  return bad;
}

// The outputs of the wavefront's problems from the last step taken (W_0 = -K_0 and P_0): only problems with keep[q] are written, NaN
// where info[q] is not 0, which is reported as info_base + info[q].
template <typename TIn, int PPW>
__device__ __forceinline__ void emit_quad16(float (*Wm)[16 * Cfg<16>::PITCH], const SolveArgs& p, const long long (&prob)[PPW],
                                            const bool (&keep)[PPW], const TIn* const (&Qp)[PPW], floatx4 (&P)[PPW],
                                            const floatx4 (&Wk)[PPW], const int (&info)[PPW], int info_base, int lane) {
  constexpr int D = 16;
  using C = Cfg<D>;
  const int i = lane & 15, g = lane >> 4, gq = g & (PPW - 1);
  // No cost on x_0.  Lane (i, g) takes row i of its problem's K_0 and P_0 for u_0 = K_0 x_0 and
  // value = x_0^T P_0 x_0; the matrices leave as one 16-byte piece per lane and problem
  long long pg = prob[0];
  int myinfo = info[0];
  bool mykeep = keep[0];
#pragma unroll
  for (int q = 1; q < PPW; ++q) {
    pg = gq == q ? prob[q] : pg;
    myinfo = gq == q ? info[q] : myinfo;
    mykeep = gq == q ? keep[q] : mykeep;
  }
  const float nanv = __builtin_nanf("");
  const float x0_m = ld1<TIn>(reinterpret_cast<const TIn*>(p.x0), pg * p.sx0 + i);
#pragma unroll
  for (int q = 0; q < PPW; ++q) {
    if (p.flags & TTC_FLAG_STAGE_COST_AT_X0)
      P[q] += 0.5f * (load_acc16<TIn>(Qp[q], i, g) + load_accT16<TIn>(Qp[q], i, g));
#pragma unroll
    for (int v = 0; v < 4; ++v) Wm[q][(4 * g + v) * C::PITCH + i] = -Wk[q][v];          // K_0, row-major
    *reinterpret_cast<floatx4*>(Wm[q] + D + i * C::PITCH + 4 * g) = P[q];                // P_0
  }
  if (g == gq) Wm[gq][i * C::PITCH + 2 * D] = x0_m;  // the first of the four skew columns
  wave_lds_sync();
  float u = 0.f, pw = 0.f;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const floatx4 kr = *reinterpret_cast<const floatx4*>(Wm[gq] + i * C::PITCH + 4 * c);
    const floatx4 pr = *reinterpret_cast<const floatx4*>(Wm[gq] + D + i * C::PITCH + 4 * c);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float xr = Wm[gq][(4 * c + v) * C::PITCH + 2 * D];
      u = __builtin_fmaf(kr[v], xr, u);
      pw = __builtin_fmaf(pr[v], xr, pw);
    }
  }
  const float val = sum16(x0_m * pw);
  if (mykeep && (PPW == 4 || g == 0)) {
    p.u0[pg * D + i] = myinfo ? nanv : u;
    if (i == 0) {
      if (p.value) p.value[pg] = myinfo ? nanv : val;
      if (p.info) p.info[pg] = myinfo ? info_base + myinfo : 0;
    }
  }
#pragma unroll
  for (int q = 0; q < PPW; ++q) {
    if (!keep[q]) continue;  // uniform over the wavefront
    const floatx4 nan4 = floatx4{nanv, nanv, nanv, nanv};
    const float* row = Wm[q] + (lane >> 2) * C::PITCH + 4 * (lane & 3);
    if (p.K0)
      *reinterpret_cast<floatx4*>(p.K0 + prob[q] * (long)D * D + 4 * lane) =
          info[q] ? nan4 : *reinterpret_cast<const floatx4*>(row);
    if (p.P0)
      *reinterpret_cast<floatx4*>(p.P0 + prob[q] * (long)D * D + 4 * lane) =
          info[q] ? nan4 : *reinterpret_cast<const floatx4*>(row + D);
  }
  wave_lds_sync();
}

// The whole backward recursion of the wavefront's PPW problems, from their terminal value matrices (PTp[q], input element
// type) to the outputs.  Step s of problem q reads A, B, R at Ap[q] + s*tA, ... and the stage cost on the state it starts
// from at Qp[q] + (s-1)*tQ; zero strides give the time-invariant problem.  Only problems with keep[q] are written;
// info = info_base + the index (1 = the step taken first) of the step whose solve broke down; returns, uniformly, whether any did.
// Measured at T = 64, kernel time, against the version that passed every operand through LDS and inverted a row per lane:
// 16 problems 195 -> 104 us, 1024: 222 -> 127 us, 8192: 1059 -> 546 us.
template <typename TIn, int PPW>
__device__ __forceinline__ bool riccati_quad(float (*Wm)[16 * Cfg<16>::PITCH], const SolveArgs& p,
                                             const long long (&prob)[PPW], const bool (&keep)[PPW], int T,
                                             const TIn* const (&Ap)[PPW], const TIn* const (&Bp)[PPW],
                                             const TIn* const (&Qp)[PPW], const TIn* const (&Rp)[PPW],
                                             const TIn* const (&PTp)[PPW], long long tA, long long tB, long long tQ,
                                             long long tR, int info_base, int tid) {
  const int lane = tid & 63, i = lane & 15, g = lane >> 4;
  int info[PPW] = {};
  int nsolve = 0;
  auto note = [&](int bad) {
    ++nsolve;
    const unsigned long long m = __ballot(bad != 0);
#pragma unroll
    for (int q = 0; q < PPW; ++q)
      if (!info[q] && ((m >> (16 * q)) & 0xFFFFull)) info[q] = nsolve;
  };
  // One problem per wavefront is the shape of batches that do not fill the chip, where nothing else hides a step's reads:
  // its matrices are requested two steps ahead (PF), into the registers of the step that has just used its own.  With four
  // problems A and B are requested one step ahead, and R and Q, which a step needs late, at its start.  Every step issues
  // the same reads (the last ones repeat what is there), so that a wait counts on exactly them.
  constexpr bool PF = PPW == 1;
  constexpr int NS = PF ? 2 : 1;
  floatx4 A[NS][PPW], B[NS][PPW], R0[NS][PPW], R1[NS][PPW], Q0[NS][PPW], Q1[NS][PPW];
  int left = T - 1, left_r = T - 1, left_q = T - 1;  // steps before the one whose reads are issued next
  long long oA = (T - 1) * tA, oB = (T - 1) * tB, oR = (T - 1) * tR, oQ = T >= 2 ? (T - 2) * tQ : 0;
  auto fetch_ab = [&](int u) {
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
      A[u][q] = load_acc16<TIn>(Ap[q] + oA, i, g);
      B[u][q] = load_acc16<TIn>(Bp[q] + oB, i, g);
    }
    if (left > 0) {
      --left;
      oA -= tA;
      oB -= tB;
    }
  };
  auto fetch_r = [&](int u) {
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
      R0[u][q] = load_acc16<TIn>(Rp[q] + oR, i, g);
      R1[u][q] = load_accT16<TIn>(Rp[q] + oR, i, g);
    }
    if (left_r > 0) {
      --left_r;
      oR -= tR;
    }
  };
  auto fetch_q = [&](int u) {  // the stage cost on the state the step starts from
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
      Q0[u][q] = load_acc16<TIn>(Qp[q] + oQ, i, g);
      Q1[u][q] = load_accT16<TIn>(Qp[q] + oQ, i, g);
    }
    if (left_q > 1) oQ -= tQ;
    --left_q;
  };
  floatx4 P[PPW], Wk[PPW];
#pragma unroll
  for (int u = 0; u < NS; ++u) {
    fetch_ab(u);
    if (PF) {
      fetch_r(u);
      fetch_q(u);
    }
  }
#pragma unroll
  for (int q = 0; q < PPW; ++q)  // P_T = Q_T
    P[q] = 0.5f * (load_acc16<TIn>(PTp[q], i, g) + load_accT16<TIn>(PTp[q], i, g));
  auto step = [&](auto U, int s) {
    constexpr int u = decltype(U)::value;
    if (!PF) {
      fetch_r(u);
      fetch_q(u);
    }
    floatx4 pn[PPW], S[PPW], Si[PPW];
    note(riccati_step16<PPW>(Wm, P, A[u], B[u], [&](int q) { return 0.5f * (R0[u][q] + R1[u][q]); },
                             [&] {
                               fetch_ab(u);
                               if (PF) fetch_r(u);
                             },
                             Wk, pn, S, Si, lane));
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
      P[q] = pn[q];
      if (s >= 1) P[q] += 0.5f * (Q0[u][q] + Q1[u][q]);
    }
    if (PF) fetch_q(u);
    symmetrise16<PPW>(P, i, g);
    wave_lds_sync();
  };
  for (int s = T - 1; s >= 0; s -= NS) {
    step(IntC<0>{}, s);
    if constexpr (NS == 2) {
      if (s == 0) break;
      step(IntC<1>{}, s - 1);
    }
  }
  emit_quad16<TIn, PPW>(Wm, p, prob, keep, Qp, P, Wk, info, info_base, lane);
  int any = 0;
#pragma unroll
  for (int q = 0; q < PPW; ++q) any |= info[q];
  return any != 0;
}

template <typename TIn, int PPW>
__global__ void __launch_bounds__(64, PPW == 4 ? 2 : 4) solve_tv_small_kernel(const TvArgs ta) {
  constexpr int D = 16;
  using C = Cfg<D>;
  static_assert(PPW == 1 || PPW == 4, "one problem or four per wavefront");
  __shared__ __attribute__((aligned(16))) float Wm[PPW][D * C::PITCH];
  const SolveArgs& p = ta.s;
  const long long nquads = (p.n + PPW - 1) / PPW;

  for (long long quad = blockIdx.x; quad < nquads; quad += gridDim.x) {
    const int tid = threadIdx.x + opaque_zero();
    long long prob[PPW];  // a ragged last quad repeats the last problem; only valid ones are written out
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
      PTp[q] = Qp[q] + (long long)(p.T - 1) * ta.tQ;  // P_T = Q_T
    }
    riccati_quad<TIn, PPW>(Wm, p, prob, valid, p.T, Ap, Bp, Qp, Rp, PTp, ta.tA, ta.tB, ta.tQ, ta.tR, 0, tid);
  }
}

}  // namespace ttc
