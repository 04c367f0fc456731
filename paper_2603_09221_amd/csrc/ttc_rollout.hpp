// Roll-out kernel of the time-invariant problem (Alg. 1, forward loop, r = 0).
#pragma once
#include "ttc_columns.hpp"
#include "ttc_common.hpp"

namespace ttc {

// ------------------------------------------------------------------------------------------------

// Matrix-vector products y = M x of a row-major d x d matrix, NTHR / d threads (adjacent lanes) to a row r = tid / TPR, each with
// its share of the columns.  A share is read into registers in one go, before anything waits for it: left to the scheduler, which
// saves registers where another part of the kernel needs many, the reads come one after the other, each with its latency (the
// loops of a time-heterogeneous backward pass 1.7 to 2.5 times as long, measured).
template <int D, typename V = floatx4>  // V: four entries as read
struct RowShare {
  static constexpr int TPR = Cfg<D>::NTHR / D;  // 2 or 4
  V v[D / TPR / 4];
  template <typename MatLoad4>  // (row, column) -> four consecutive entries
  __device__ __forceinline__ void load(MatLoad4&& row4, int tid) {
    const int r = tid / TPR, c0 = (tid % TPR) * (D / TPR);
#pragma unroll
    for (int c = 0; c < D / TPR / 4; ++c) v[c] = row4(r, c0 + 4 * c);
  }
  __device__ __forceinline__ float dot(const float* xs, int tid) const {
    const int c0 = (tid % TPR) * (D / TPR);
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < D / TPR / 4; ++c) {
      const floatx4 x = *reinterpret_cast<const floatx4*>(xs + c0 + 4 * c);
      const floatx4 m = widen(v[c]);
      s += m[0] * x[0] + m[1] * x[1] + m[2] * x[2] + m[3] * x[3];
    }
    return share_sum(s);
  }
  // the sum over the row's threads, in all of them
  static __device__ __forceinline__ float share_sum(float s) {
    if constexpr (TPR >= 2)
      s += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(s), 0xB1, 0xF, 0xF, false));  // quad_perm [1,0,3,2]
    if constexpr (TPR >= 4)
      s += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(s), 0x4E, 0xF, 0xF, false));  // quad_perm [2,3,0,1]
    static_assert(TPR <= 4, "a row's threads are within a quad");
    return s;
  }
};
template <int D, typename TM>
using RowShareOf = RowShare<D, decltype(read4((const TM*)nullptr, 0))>;
template <int D, typename TM>
__device__ __forceinline__ auto rows_of(const TM* M) {
  return [M](int r, int c4) { return read4(M, (long)r * D + c4); };
}
template <int D>
__device__ __forceinline__ auto rows_in_lds(const float* M) {
  return [M](int r, int c4) { return *reinterpret_cast<const floatx4*>(M + r * Cfg<D>::PITCH + c4); };
}

// The product at once, with M in LDS (row pitch PITCH).
template <int D>
__device__ __forceinline__ float matvec_row_lds(const float* M, const float* xs, int tid) {
  RowShare<D> m;
  m.load(rows_in_lds<D>(M), tid);
  return m.dot(xs, tid);
}

// Backward sweep of rollout_kernel for a problem whose R + B^T P B is not positive definite everywhere (a stage cost that is
// not positive semidefinite): the value matrices P_T .. P_1 one step at a time in the re-based form of the reverse
// symplectic factor, whose solve is pivoted and asks for nothing but a non-singular matrix,
//     M_t = (I + P_{t+1} G)^{-1} P_{t+1} A,   K_t = -(R^{-1} B^T) M_t,   P_t = Q + A^T M_t.
// wsC: 3 d x d of workspace; the gains go to wsK.  Returns info: 1 = R, then a step each.
template <int D, typename TIn>
__device__ __forceinline__ int rollout_pivoted_sweep(float* W, SolveScratch<D>& S, int T, const TIn* Ap, const TIn* Bp,
                                                     const TIn* Qp, const TIn* Rp, const TIn* QTp, float* wsC, float* wsK,
                                                     int tid) {
  using C = Cfg<D>;
  const int lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
  float* const WL = W;
  float* const WR = W + D;
  int info = 0, nsolve = 0;
  floatx4 acc[C::RB][C::NT];

  // ---- setup: X = R^{-1} B^T, G = B X; row blocks of G, X, A^T to the workspace
  load_half<D, TIn, false>(WL, Rp, tid);
  load_half<D, TIn, false>(WR, Bp, tid);
  __syncthreads();
  symmetrise_half<D>(WL, tid);
  transpose_half<D>(WR, w, i, g);              // RHS = B^T
  ++nsolve;
  if (lds_solve<D, 7, false>(W, S, tid) && !info) info = nsolve;  // R is positive definite: no pivot search
  {
    float c[C::RB][C::KS];
    load_aop_lds<D>(WR, c, w, i, g);
    store_aop_ws<D>(wsC + 1 * D * D, c, tid);
    load_aop_global<D, TIn>(Bp, c, w, i, g);
    zero_acc<D>(acc);
    gemm_acc<D>(acc, c, WR, i, g);
    store_rows<D>(WL, acc, w, i, g);
    __syncthreads();
    symmetrise_half<D>(WL, tid);
    __syncthreads();
    load_aop_lds<D>(WL, c, w, i, g);
    store_aop_ws<D>(wsC + 0 * D * D, c, tid);
#pragma unroll
    for (int rb = 0; rb < C::RB; ++rb)
#pragma unroll
      for (int k = 0; k < C::KS; ++k)
        c[rb][k] = ld1<TIn>(Ap, (long)(16 * (k / 4) + 4 * g + (k % 4)) * D + 16 * (C::RB * w + rb) + i);
    store_aop_ws<D>(wsC + 2 * D * D, c, tid);
  }
  __syncthreads();
  load_half<D, TIn, false>(WR, QTp, tid);
  __syncthreads();
  symmetrise_half<D>(WR, tid);
  __syncthreads();

  // ---- backward sweep (the constant row blocks are read again for every product: held in registers, they would cost the
  // sweep that almost every problem takes)
  auto times = [&](int k) {  // acc += (G, X or A^T) * the right half
    float c[C::RB][C::KS];
    load_aop_ws<D>(wsC + k * D * D, c, tid, opaque_zero());
    gemm_acc<D>(acc, c, WR, i, g);
  };
  for (int t = T - 1; t >= 0; --t) {
    eye_acc<D>(acc, w, i, g);
    times(0);                         // (I + P G)^T
    store_rows_T<D>(WL, acc, w, i, g);
    zero_acc<D>(acc);
    times(2);                         // (P A)^T
    __syncthreads();
    store_rows_T<D>(WR, acc, w, i, g);
    __syncthreads();
    ++nsolve;
    if (lds_solve<D>(W, S, tid) && !info) info = nsolve;
    zero_acc<D>(acc);
    times(1);                         // -K_t
#pragma unroll
    for (int rb = 0; rb < C::RB; ++rb) {
#pragma unroll
      for (int cc = 0; cc < C::NT; ++cc) acc[rb][cc] = -acc[rb][cc];
      write_rows_global<D>(wsK + (long)t * D * D, acc[rb], C::RB * w + rb, i, g);
    }
    if (t >= 1) {
#pragma unroll
      for (int rb = 0; rb < C::RB; ++rb)
#pragma unroll
        for (int cc = 0; cc < C::NT; ++cc)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const long row = 16 * (C::RB * w + rb) + 4 * g + v, col = tile_col<D>(cc, i);
            acc[rb][cc][v] = 0.5f * (ld1<TIn>(Qp, row * D + col) + ld1<TIn>(Qp, col * D + row));
          }
      times(2);                         // P_t = Q + A^T M_t
      __syncthreads();
      store_rows<D>(WR, acc, w, i, g);
      __syncthreads();
      symmetrise_half<D>(WR, tid);
      __syncthreads();
    }
  }
  return info;
}

// Roll-out kernel (Alg. 1 with r = 0).  Backward sweep: the recursion of Prop. 3.1 as ttc_lqr_solve_tv runs it, with the
// same matrices in every step, the gains to the workspace; forward sweep: u_t = K_t x_t, x_{t+1} = A x_t + B u_t and the
// cost, A and B read from LDS.  R is factored once for its report.
// Every step needs R and Q as their symmetric parts: these are formed once and kept as the registers hold them (read anew in
// every step, two elements apart for bfloat16, they made it slower than the pivoted sweep's at d = 128: 24 steps of 256
// problems 1.98 -> 2.10 ms, with the kept ones 2.01).
// Against the pivoted sweep for every problem and all five matrices of a forward step from memory: d = 64, T = 8, 4096
// problems 1.94 -> 1.38 ms; d = 32, 8192 problems 0.80 -> 0.47 ms; d = 128, 1024 problems 3.01 -> 2.74 ms.
template <int D, typename TIn>
__global__ void __launch_bounds__(Cfg<D>::NTHR, TTC_COLS_WAVES(D)) rollout_kernel(const RolloutArgs p) {
  using C = Cfg<D>;
  __shared__ __attribute__((aligned(16))) float W[C::PAIR];
  __shared__ __attribute__((aligned(16))) SolveScratch<D> S;
  __shared__ float s_red[C::NW];
  // the forward sweep's vectors, where the pivoted sweep has a factor (at d = 32 their 384 bytes would cost the twelfth workgroup of a
  // compute unit: T = 8, 8192 problems 0.53 against 0.38 ms)
  static_assert(sizeof(S.Linv) >= 3 * D * sizeof(float), "");
  float* const s_x = S.Linv[0];
  float* const s_u = s_x + D;
  float* const s_xn = s_u + D;

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  float* const WL = W;
  float* const WR = W + D;
  // symmetric parts of R and Q, in register layout (the pivoted sweep: G, X, A^T)
  float* const wsC = p.ws + (long)blockIdx.x * (p.T + 3) * D * D;
  float* const wsK = wsC + 3 * D * D;                              // K_0 .. K_{T-1}, row-major

  for (long long prob = blockIdx.x; prob < p.n; prob += gridDim.x) {
    const TIn* Ap = reinterpret_cast<const TIn*>(p.A) + prob * p.sA;
    const TIn* Bp = reinterpret_cast<const TIn*>(p.B) + prob * p.sB;
    const TIn* Qp = reinterpret_cast<const TIn*>(p.Q) + prob * p.sQ;
    const TIn* Rp = reinterpret_cast<const TIn*>(p.R) + prob * p.sR;
    const TIn* QTp = p.QT ? reinterpret_cast<const TIn*>(p.QT) + prob * p.sQT : Qp;
    const TIn* x0p = reinterpret_cast<const TIn*>(p.x0) + prob * p.sx0;
    int info = 0;
    {
      const int tb = tid + opaque_zero(), lane = tb & 63, w = uniform(tb >> 6), i = lane & 15, g = lane >> 4;
      {
        Cols<D> r;
        floatx4 none[C::NT][1];  // no right-hand sides
        zero_cols<D>(r);
        add_sym_cols<D, TIn>(Rp, r, w, i, g);
        keep_cols<D>(wsC, r, tb);
        info = solve_cols<D, 0>(WR, r, none, w, lane);
      }
      __syncthreads();
      if (!info) {
        load_half<D, TIn, false>(WR, QTp, tb);  // P_T = Q_T
        __syncthreads();
        symmetrise_half<D>(WR, tb);
        __syncthreads();
        {
          Cols<D> q;
          zero_cols<D>(q);
          add_sym_cols<D, TIn>(Qp, q, w, i, g);
          keep_cols<D>(wsC + D * D, q, tb);
        }
        int t = p.T - 1;
        for (; t >= 0; --t) {
          Cols<D> wk, pn;
          const int tk = tb + opaque_zero();
          if (riccati_step_with<D, TIn>(
                  W, Ap, Bp, Rp, [&](Cols<D>& s, int, int, int) { add_kept_cols<D>(wsC, s, tk); }, wk, pn, tb))
            break;
          store_cols<D, -1>(wsK + (long)t * D * D, D, wk, w, i, g);  // K_t
          if (t >= 1)
            next_value_matrix_with<D>(W, [&](Cols<D>& m, int, int, int) { add_kept_cols<D>(wsC + D * D, m, tk); }, pn, tb);
        }
        if (t >= 0) {
          __syncthreads();
          info = rollout_pivoted_sweep<D, TIn>(W, S, p.T, Ap, Bp, Qp, Rp, QTp, wsC, wsK, tb);
        }
      }
    }
    __syncthreads();
    load_half<D, TIn, false>(WL, Ap, tid);
    load_half<D, TIn, false>(WR, Bp, tid);
    __syncthreads();  // gains visible to the whole workgroup

    // ---- forward sweep; R and Q stay in registers, the next gain is on its way
    const int r = tid / (C::NTHR / D), part = tid % (C::NTHR / D);
    RowShare<D> Kr;
    RowShareOf<D, TIn> Rr, Qr;
    Kr.load(rows_of<D, float>(wsK), tid);
    Rr.load(rows_of<D, TIn>(Rp), tid);
    Qr.load(rows_of<D, TIn>(p.T == 1 && !(p.flags & TTC_FLAG_STAGE_COST_AT_X0) ? QTp : Qp), tid);
    if (tid < D) s_x[tid] = ld1<TIn>(x0p, tid);
    __syncthreads();
    float cpart = 0.f;
    if (p.flags & TTC_FLAG_STAGE_COST_AT_X0) {
      const float qx = Qr.dot(s_x, tid);
      if (part == 0) cpart += s_x[r] * qx;
      if (p.T == 1) Qr.load(rows_of<D, TIn>(QTp), tid);
    }
    if (p.X && tid < D) p.X[prob * (long)(p.T + 1) * D + tid] = s_x[tid];
    for (int t = 0; t < p.T; ++t) {
      const float u = Kr.dot(s_x, tid);
      if (t + 1 < p.T) Kr.load(rows_of<D, float>(wsK + (long)(t + 1) * D * D), tid);
      const float ax = matvec_row_lds<D>(WL, s_x, tid);
      if (part == 0) s_u[r] = u;
      lds_barrier();
      const float ru = Rr.dot(s_u, tid);
      const float xn = ax + matvec_row_lds<D>(WR, s_u, tid);
      if (part == 0) {
        cpart += u * ru;
        s_xn[r] = xn;
        p.U[(prob * p.T + t) * (long)D + r] = info ? __builtin_nanf("") : u;
        if (p.X) p.X[(prob * (p.T + 1) + t + 1) * (long)D + r] = info ? __builtin_nanf("") : xn;
      }
      lds_barrier();
      const float qx = Qr.dot(s_xn, tid);
      if (t == p.T - 2 && QTp != Qp) Qr.load(rows_of<D, TIn>(QTp), tid);
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

}  // namespace ttc
