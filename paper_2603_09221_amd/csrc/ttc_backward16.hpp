// The backward pass of the layer (ttc_backward.hpp has the method) at d = 16: a workgroup of one wavefront per problem,
// register to register.  A call at the sizes of the paper's benchmark is bound by the latency of its three serial sweeps
// over the horizon, so a step does as little as possible in series: the recursion is riccati_step16 (ttc_tv.hpp); a
// closed-loop step is two dependent products of four matrix instructions, in two halves (dot16), for the primal and the
// dual trajectory together (a state is a 16 x 16 operand with the primal in column 0 and the dual in column 1); a co-state
// step is one, beside which the four gradients of the step before, rank-2 outer products, are one matrix instruction each.
// The matrices of a step are requested one step ahead.  Measured, kernel time at T = 64, against backward_kernel at d = 16
// (operands through LDS, a workgroup barrier per exchange): 16 problems 417 -> 173 us, 1024: 647 -> 280 us, 2048: 857 -> 440
// us; at 1024 problems and up it is the traffic, some 14 KB per problem and step, that counts (3.5 TB/s).
#pragma once
#include "ttc_tv.hpp"

namespace ttc {

// L R in two halves of the contraction that are added at the end: a sum of sixteen terms one after the other, on top of
// another such sum, carries more rounding than the tree a matrix-vector product by lanes adds up (states, controls and
// co-states are such products all through the horizon).
__device__ __forceinline__ floatx4 dot16(const floatx4& a, const floatx4& b) {
  floatx4 e = floatx4{0.f, 0.f, 0.f, 0.f}, o = e;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    e = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t], b[t], e, 0, 0, 0);
    o = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t + 2], b[t + 2], o, 0, 0, 0);
  }
  return e + o;
}

// PAST: the gradients of the steps are written past the caches (use_past_caches, ttc_api.hip).  A template argument: of a
// branch around the two stores the compiler makes one plain store.
template <bool PAST>
__device__ __forceinline__ void store_gradient16(float* p, const floatx4& v) {
  if constexpr (PAST)
    __builtin_nontemporal_store(v, reinterpret_cast<floatx4*>(p));
  else
    *reinterpret_cast<floatx4*>(p) = v;
}

template <typename TIn, bool PAST>
__global__ void __launch_bounds__(64, 4) backward16_kernel(const BackwardArgs ba) {
  constexpr int D = 16, DD = D * D;
  using C = Cfg<D>;
  __shared__ __attribute__((aligned(16))) float Wm[1][D * C::PITCH];
  __shared__ __attribute__((aligned(16))) float s_lam[2][D];  // co-states, primal and dual
  const RolloutArgs& p = ba.r;
  const int T = p.T;
  float* const wsK = p.ws + (long)blockIdx.x * ((long)(T - 1) * DD + 6L * (T + 1) * D);  // K_1 .. K_{T-1}, row-major
  float* const traj = wsK + (long)(T - 1) * DD;  // step s at 64 s: x, xt, u, ut
  const float nanv = __builtin_nanf("");

  for (long long prob = blockIdx.x; prob < p.n; prob += gridDim.x) {
    const int lane = threadIdx.x + opaque_zero(), i = lane & 15, g = lane >> 4;
    const TIn* Ap = reinterpret_cast<const TIn*>(p.A) + prob * p.sA;
    const TIn* Bp = reinterpret_cast<const TIn*>(p.B) + prob * p.sB;
    const TIn* Qp = reinterpret_cast<const TIn*>(p.Q) + prob * p.sQ;
    const TIn* Rp = reinterpret_cast<const TIn*>(p.R) + prob * p.sR;
    const TIn* x0p = reinterpret_cast<const TIn*>(p.x0) + prob * p.sx0;
    // the terminal cost: a separate matrix for time-invariant problems that give one, else Q of the last step
    const TIn* QTp = p.QT ? reinterpret_cast<const TIn*>(p.QT) + prob * p.sQT : Qp + (long long)(T - 1) * ba.tQ;
    const float* gp = ba.g + prob * ba.sg;
    int info = 0;

    // ---- backward recursion (Prop. 3.1): K_{T-1} .. K_1 to the workspace; the last step (s = 0) stays in registers
    floatx4 P[1], W[1], S[1], Si[1];
    floatx4 A[2][1], B[2][1], R0[2], R1[2], Q0[2], Q1[2];
    // a step's matrices are requested two steps ahead, into the registers of the step that has just used its own; every
    // step issues the same reads (the last ones repeat), so that a wait counts on exactly them
    auto fetch_abr = [&](int u, int s) {
      s = s < 0 ? 0 : s;
      A[u][0] = load_acc16<TIn>(Ap + (long long)s * ba.tA, i, g);
      B[u][0] = load_acc16<TIn>(Bp + (long long)s * ba.tB, i, g);
      R0[u] = load_acc16<TIn>(Rp + (long long)s * ba.tR, i, g);
      R1[u] = load_accT16<TIn>(Rp + (long long)s * ba.tR, i, g);
    };
    auto fetch_q = [&](int u, int s) {  // the stage cost on the state step s starts from
      s = s < 1 ? 1 : s;
      Q0[u] = load_acc16<TIn>(Qp + (long long)(s - 1) * ba.tQ, i, g);
      Q1[u] = load_accT16<TIn>(Qp + (long long)(s - 1) * ba.tQ, i, g);
    };
    fetch_abr(0, T - 1);
    fetch_q(0, T - 1);
    fetch_abr(1, T - 2);
    fetch_q(1, T - 2);
    P[0] = 0.5f * (load_acc16<TIn>(QTp, i, g) + load_accT16<TIn>(QTp, i, g));
    auto step = [&](auto U, int s) {
      constexpr int u = decltype(U)::value;
      floatx4 pn[1];
      const int bad = riccati_step16<1, true>(Wm, P, A[u], B[u], [&](int) { return 0.5f * (R0[u] + R1[u]); },
                                        [&] { fetch_abr(u, s - 2); }, W, pn, S, Si, lane);
      if (__any(bad) && !info) info = T - s;
      if (s >= 1) {
#pragma unroll
        for (int v = 0; v < 4; ++v) wsK[(long)(s - 1) * DD + (unsigned)(64 * g + i) + 16 * v] = -W[0][v];
        P[0] = pn[0] + 0.5f * (Q0[u] + Q1[u]);
        fetch_q(u, s - 2);
        symmetrise16<1>(P, i, g);
      }
    };
    for (int s = T - 1; s >= 0; s -= 2) {
      step(IntC<0>{}, s);
      if (s == 0) break;
      step(IntC<1>{}, s - 1);
    }

    // ---- first controls: u_0 = -W_0 x_0 and ut_0 = -S_0^{-1} g, the latter refined once with S_0
    floatx4 X[1], U[1];
    {
      floatx4 eye[1], WT[1], G[1], y[1], neg[1];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        eye[0][v] = (4 * g + v == i) ? 1.f : 0.f;
        X[0][v] = i == 0 ? ld1<TIn>(x0p, 4 * g + v) : 0.f;
        G[0][v] = i == 1 ? gp[4 * g + v] : 0.f;
      }
      zero16<1>(WT);
      mul16<1>(WT, W, eye);  // W_0^T in the accumulator layout: the A operand of W_0
      zero16<1>(y);
      mul16<1>(y, Si, G);
      neg[0] = -S[0];
      floatx4 res[1] = {G[0]};
      mul16<1>(res, neg, y);
      mul16<1>(y, Si, res);
      mul16<1>(y, WT, X);
      U[0] = -y[0];
    }
    __syncthreads();  // the gains are visible to every lane

    // ---- both closed loops forward (Alg. 1)
    {
      floatx4 An = load_accT16<TIn>(Ap, i, g), Bn = load_accT16<TIn>(Bp, i, g), Kn = floatx4{0.f, 0.f, 0.f, 0.f};
      for (int s = 0; s < T; ++s) {
        const floatx4 Ac = An, Bc = Bn, Kc = Kn;
        const int sn = s + 1 < T ? s + 1 : s;
        An = load_accT16<TIn>(Ap + (long long)sn * ba.tA, i, g);
        Bn = load_accT16<TIn>(Bp + (long long)sn * ba.tB, i, g);
        if (T > 1) Kn = *reinterpret_cast<const floatx4*>(wsK + (long)(sn - 1) * DD + (unsigned)(i * D + 4 * g));  // K_{s+1}
        if (s >= 1) U[0] = dot16(Kc, X[0]);
        const floatx4 Ax = dot16(Ac, X[0]);
        if (i < 2) {
          *reinterpret_cast<floatx4*>(traj + 64L * s + 16 * i + 4 * g) = X[0];
          *reinterpret_cast<floatx4*>(traj + 64L * s + 32 + 16 * i + 4 * g) = U[0];
        }
        X[0] = Ax + dot16(Bc, U[0]);
      }
      if (i < 2) *reinterpret_cast<floatx4*>(traj + 64L * T + 16 * i + 4 * g) = X[0];
    }
    __syncthreads();  // the trajectories are visible to every lane

    // ---- co-states backward (Alg. 2) and the gradients of every step.  A gradient is formed transposed, so that a lane
    // ends with four consecutive entries of a row: entry (k, i) of the two operands is vector k of a pair, k < 2.
    floatx4 L[1], sA = floatx4{0.f, 0.f, 0.f, 0.f}, sB = sA, sQ = sA, sR = sA, sQT = sA;
    {
      floatx4 Qs[1] = {0.5f * (load_acc16<TIn>(QTp, i, g) + load_accT16<TIn>(QTp, i, g))};
      L[0] = dot16(Qs[0], X[0]);  // lam_T = Q_T x_T
    }
    const bool two = g < 2;
    auto vec = [&](int s, int off, int k) { return traj[64L * s + (unsigned)(off + 16 * k + i)]; };
    float xt_own = two ? vec(T, 0, g & 1) : 0.f, xt_other = two ? vec(T, 0, 1 - (g & 1)) : 0.f;  // x_{s+1}: vector g, the other
    floatx4 An = load_acc16<TIn>(Ap + (long long)(T - 1) * ba.tA, i, g), Qn0, Qn1, Xs;
    float x_own, x_other, u_own, u_other;
    auto fetch = [&](int s) {  // what step s's gradients and the co-state of its start need
      x_own = vec(s, 0, g & 1);
      x_other = vec(s, 0, 1 - (g & 1));
      u_own = vec(s, 32, g & 1);
      u_other = vec(s, 32, 1 - (g & 1));
      const int sq = s >= 1 ? s - 1 : 0;
      Qn0 = load_acc16<TIn>(Qp + (long long)sq * ba.tQ, i, g);
      Qn1 = load_accT16<TIn>(Qp + (long long)sq * ba.tQ, i, g);
      Xs = *reinterpret_cast<const floatx4*>(traj + 64L * s + (unsigned)(16 * (i & 1) + 4 * g));
    };
    fetch(T - 1);
    for (int s = T - 1; s >= 0; --s) {
      if (i < 2) *reinterpret_cast<floatx4*>(&s_lam[i][4 * g]) = L[0];  // lam_{s+1}
      wave_lds_sync();
      const float lam = two ? s_lam[g & 1][i] : 0.f;
      const floatx4 Ac = An, Qs = 0.5f * (Qn0 + Qn1), Xc = Xs;
      // an outer product has two terms: groups 2 and 3 are zero
      const float xo = two ? x_own : 0.f, xx = two ? x_other : 0.f, uo = two ? u_own : 0.f, ux = two ? u_other : 0.f;
      const int sn = s >= 1 ? s - 1 : 0;
      An = load_acc16<TIn>(Ap + (long long)sn * ba.tA, i, g);
      fetch(sn);
      floatx4 Ln = dot16(Ac, L[0]);  // A_s^T lam_{s+1}
      if (s >= 1) Ln += dot16(Qs, Xc);
      // a step's gradients are formed on their own and then added to the sum
      const floatx4 none = floatx4{0.f, 0.f, 0.f, 0.f};
      const floatx4 dA = __builtin_amdgcn_mfma_f32_16x16x4f32(xx, lam, none, 0, 0, 0);  // transposed: xt lam^T + x lamt^T
      const floatx4 dB = __builtin_amdgcn_mfma_f32_16x16x4f32(ux, lam, none, 0, 0, 0);
      const floatx4 dR = __builtin_amdgcn_mfma_f32_16x16x4f32(0.5f * ux, uo, none, 0, 0, 0);
      const floatx4 dQ = __builtin_amdgcn_mfma_f32_16x16x4f32(0.5f * xt_other, xt_own, none, 0, 0, 0);
      if (!ba.sum_steps) sA = sB = sQ = sR = none;
      sA += dA;
      sB += dB;
      sR += dR;
      if (ba.gQT && s == T - 1) sQT += dQ;
      else sQ += dQ;
      if (!ba.sum_steps) {
        const long long o = (prob * T + s) * DD + i * D + 4 * g;
        const floatx4 nan4 = floatx4{nanv, nanv, nanv, nanv};
        store_gradient16<PAST>(ba.gA + o, info ? nan4 : sA);
        store_gradient16<PAST>(ba.gB + o, info ? nan4 : sB);
        store_gradient16<PAST>(ba.gQ + o, info ? nan4 : sQ);
        store_gradient16<PAST>(ba.gR + o, info ? nan4 : sR);
      }
      xt_own = xo;
      xt_other = xx;
      L[0] = Ln;
      wave_lds_sync();
    }
    if (ba.sum_steps) {
      const long long o = prob * DD + i * D + 4 * g;
      const floatx4 nan4 = floatx4{nanv, nanv, nanv, nanv};
      *reinterpret_cast<floatx4*>(ba.gA + o) = info ? nan4 : sA;
      *reinterpret_cast<floatx4*>(ba.gB + o) = info ? nan4 : sB;
      *reinterpret_cast<floatx4*>(ba.gQ + o) = info ? nan4 : sQ;
      *reinterpret_cast<floatx4*>(ba.gR + o) = info ? nan4 : sR;
      if (ba.gQT) *reinterpret_cast<floatx4*>(ba.gQT + o) = info ? nan4 : sQT;
    }
    if (i == 1) {
#pragma unroll
      for (int v = 0; v < 4; ++v) ba.gx0[prob * D + 4 * g + v] = info ? nanv : L[0][v];
    }
    if (lane == 0 && p.info) p.info[prob] = info;
    __syncthreads();  // the workspace slot is free for the next problem
  }
}

}  // namespace ttc
