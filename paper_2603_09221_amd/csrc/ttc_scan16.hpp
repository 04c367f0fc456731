// The tree over the horizon (ttc_scan.hpp) at d = 16: four elements or applications per wavefront (compositions run one to a
// wavefront, from register to register: Composition16).
//
// At d = 16 an element fills a quarter of a wavefront and its dense solve is most of its instructions; as in the d = 16
// solve kernels (ttc_small.hpp) a workgroup of one wavefront takes four items at a time, forms the products item by item
// on the matrix cores and runs the four dense solves side by side, lane 16q + r owning row r of item q.  The arithmetic,
// the workspace layout and the order of the rounds are those of the kernels of ttc_scan.hpp; a ragged last group of four
// repeats its last item and writes it once.
#pragma once
#include "ttc_scan.hpp"
#include "ttc_small.hpp"

namespace ttc {

constexpr int SCAN16_PPW = 4;

template <typename TIn>
__global__ void __launch_bounds__(64, 2) scan_leaf16_kernel(const ScanArgs a) {
  constexpr int D = 16, PPW = SCAN16_PPW;
  using C = Cfg<D>;
  __shared__ __attribute__((aligned(16))) float Wm[PPW][D * C::PITCH];
  const SolveArgs& p = a.tv.s;
  const long long items = p.n * p.T;
  const long long nquads = (items + PPW - 1) / PPW;
  for (long long quad = blockIdx.x; quad < nquads; quad += gridDim.x) {
    const int tid = threadIdx.x + opaque_zero(), lane = tid & 63, i = lane & 15, g = lane >> 4;
    constexpr int w = 0;
    float* const Wmine = Wm[g & (PPW - 1)];
    bool valid[PPW], terminal[PPW];
    const TIn *Ap[PPW], *Rp[PPW];
    float* gA[PPW];
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
      valid[q] = quad * PPW + q < items;
      const long long item = valid[q] ? quad * PPW + q : items - 1;
      const long long prob = item / p.T;
      const int k = (int)(item % p.T);
      terminal[q] = k == p.T - 1;
      // the terminal element has no step of its own: it reads the last step's matrices (in bounds) and writes zeros
      const int s = terminal[q] ? k : k + 1;
      Ap[q] = reinterpret_cast<const TIn*>(p.A) + prob * p.sA + (long long)s * a.tv.tA;
      Rp[q] = reinterpret_cast<const TIn*>(p.R) + prob * p.sR + (long long)s * a.tv.tR;
      const TIn* Bp = reinterpret_cast<const TIn*>(p.B) + prob * p.sB + (long long)s * a.tv.tB;
      const TIn* Qp = reinterpret_cast<const TIn*>(p.Q) + prob * p.sQ + (long long)k * a.tv.tQ;  // Q[k] = Q_{s-1}
      gA[q] = a.ws + item * 3 * D * D;
      load_half<D, TIn, false>(Wm[q], Qp, tid);
      load_half<D, TIn, true>(Wm[q] + D, Bp, tid);  // right-hand sides: B^T
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PPW; ++q) symmetrise_half<D>(Wm[q], tid);
    __syncthreads();
    floatx4 acc[PPW][C::RB][C::NT];
    float cB[PPW][C::RB][C::KS];
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
      if (valid[q]) store_half_global<D>(gA[q] + 2 * D * D, Wm[q], tid);  // H = sym(Q[k])
      load_aopT_lds<D>(Wm[q] + D, cB[q], w, i, g);                        // rows of B = columns of B^T
      load_rows_input<D, TIn>(Ap[q], acc[q], w, i, g);
      if (terminal[q]) zero_acc<D>(acc[q]);
      if (valid[q]) write_rows_global<D>(gA[q], acc[q], w, i, g);         // A
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PPW; ++q) load_half<D, TIn, false>(Wm[q], Rp[q], tid);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PPW; ++q) symmetrise_half<D>(Wm[q], tid);
    __syncthreads();
    const unsigned long long badm = __ballot(solve_rows16<false>(Wmine, lane) != 0);  // right halves: X = R^{-1} B^T
#pragma unroll
    for (int q = 0; q < PPW; ++q) zero_acc<D>(acc[q]);
    gemm_acc_quad<PPW>(acc, cB, Wm, D, i, g);  // G = B X
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
      if (!valid[q]) continue;
      const bool bad = !terminal[q] && ((badm >> (16 * q)) & 0xFFFFull) != 0;
      if (terminal[q]) zero_acc<D>(acc[q]);
      if (bad) poison<D>(acc[q]);
      write_rows_global<D>(gA[q] + D * D, acc[q], w, i, g);
      if (bad) write_rows_global<D>(gA[q] + 2 * D * D, acc[q], w, i, g);  // the breakdown reaches P_1 whatever follows
    }
    __syncthreads();
  }
}

// A composition (scan_compose has the algebra) from register to register, by one wavefront: the accumulator layout of a matrix (lane (i, g) holds M[4g + v][i])
// is the right operand of a product and the left operand of the transpose's, a row of four entries a lane the left operand of the
// matrix, and I + G1 H2 is formed transposed so that its inverse comes as a left operand.
struct Composition16 {
  floatx4 H2, G1, A2, A1, H, G, n;  // n: (I + G1 H2)^T
  __device__ __forceinline__ void load(const float* e1, const float* e2, int lane) {
    constexpr int DD = 256;
    const int i = lane & 15, g = lane >> 4;
    auto rows = [&](const float* m) { return *reinterpret_cast<const floatx4*>(m + 16 * i + 4 * g); };
    H2 = rows(e2 + 2 * DD);  // (G and H are symmetric)
    G1 = rows(e1 + DD);
    A2 = rows(e2);
#pragma unroll
    for (int v = 0; v < 4; ++v) A1[v] = e1[64 * g + 16 * v + i];
    H = rows(e1 + 2 * DD);
    G = rows(e2 + DD);
#pragma unroll
    for (int v = 0; v < 4; ++v) n[v] = 4 * g + v == i ? 1.f : 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) n = __builtin_amdgcn_mfma_f32_16x16x4f32(H2[t], G1[t], n, 0, 0, 0);  // I + H2 G1 = (I + G1 H2)^T
  }
  // x <- the inverse of n, without a search for pivots.  False where that is not safe (max |I + G1 H2| above 24, a pivot below 1/4,
  // anything not finite; ttc_squaring.hpp has what these limits rest on).
  // W: 16 x PITCH floats of LDS.
  __device__ __forceinline__ bool invert_in_order(floatx4& x, float* W, int lane) const {
    uint32_t big = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const uint32_t b = __float_as_uint(n[v]) & 0x7FFFFFFFu;
      big = b > big ? b : big;
    }
    const float mu = __uint_as_float(wave_max_u32(big));
    if (!(mu <= 24.f)) return false;
    x = n;
    return !invert_spread16(x, W, Cfg<16>::PITCH, lane, 0.25f);
  }
  // The element, x the inverse of n; into e1.
  __device__ __forceinline__ void finish(const floatx4& x, float* e1, int lane, bool bad) {
    constexpr int DD = 256;
    const int i = lane & 15, g = lane >> 4;
    const floatx4 z = floatx4{0.f, 0.f, 0.f, 0.f};
    floatx4 X1 = z, Y = z, A = z, V = z, Z = z;
#define TTC_STEP(c, a, b) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t], b[t], c, 0, 0, 0)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      TTC_STEP(X1, x, A1);  // M A1
      TTC_STEP(Y, x, G1);   // M G1, symmetric
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      TTC_STEP(A, A2, X1);  // A2 M A1
      TTC_STEP(V, H2, X1);  // H2 M A1
      TTC_STEP(Z, Y, A2);   // M G1 A2^T
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      TTC_STEP(H, A1, V);  // H1 + A1^T H2 M A1
      TTC_STEP(G, A2, Z);  // G2 + A2 M G1 A2^T
    }
#undef TTC_STEP
    if (bad) H = floatx4{__builtin_nanf(""), __builtin_nanf(""), __builtin_nanf(""), __builtin_nanf("")};
#pragma unroll
    for (int v = 0; v < 4; ++v) e1[64 * g + 16 * v + i] = A[v];
    *reinterpret_cast<floatx4*>(e1 + DD + 16 * i + 4 * g) = G;
    *reinterpret_cast<floatx4*>(e1 + 2 * DD + 16 * i + 4 * g) = H;
  }
};

// One round of pairwise compositions at d = 16, one to a wavefront.  A round with few items is a composition's latency, mostly the
// inverse's; with many it is bound by the inverse's instructions.  Where elimination in order is not safe (control that costs a hundredth,
// say) only the inverse passes through LDS, for the pivoted solve; all of such a composition through LDS took 10 % longer than one without the
// attempt.  T = 2048, all rounds, us a call, 16 problems: 150 in order, 200 pivoted (with four compositions side by side and all of them
// pivoted and through LDS 197); one problem 68, 90 (97).  1024 problems, T = 64: 235, 301 (284).
__global__ void __launch_bounds__(64) scan_combine16_kernel(const ScanArgs a) {
  using C = Cfg<16>;
  __shared__ __attribute__((aligned(16))) float W[16 * C::PITCH];
  __shared__ __attribute__((aligned(16))) SolveScratch<16> S;
  const SolveArgs& p = a.tv.s;
  const int st = a.stride;
  const long long per = (p.T - st + 2LL * st - 1) / (2LL * st);  // pairs per problem in this round
  const long long items = p.n * per;
  for (long long item = blockIdx.x; item < items; item += gridDim.x) {
    const int lane = threadIdx.x + opaque_zero(), i = lane & 15, g = lane >> 4;
    float* const e1 = a.ws + ((item / per) * p.T + (item % per) * 2 * st) * 3 * 256;
    Composition16 c;
    floatx4 x;
    c.load(e1, e1 + (long long)st * 3 * 256, lane);
    bool bad = false;
    if (__builtin_expect(!c.invert_in_order(x, W, lane), 0)) {  // with a search for pivots
      float* const row = W + i * C::PITCH + 4 * g;
      *reinterpret_cast<floatx4*>(row) = c.n;  // (a row of I + G1 H2)
      set_half_identity<16>(W + 16, lane);
      __syncthreads();
      bad = lds_solve<16>(W, S, lane) != 0;
      x = *reinterpret_cast<const floatx4*>(row + 16);
      __syncthreads();
    }
    c.finish(x, e1, lane, bad);
  }
}

// one level of the down-sweep, four elements per wavefront: P <- H_e + A_e^T (I + P G_e)^{-1} P A_e into the element's H
__global__ void __launch_bounds__(64, 2) scan_apply16_kernel(const ScanArgs a) {
  constexpr int D = 16, PPW = SCAN16_PPW;
  using C = Cfg<D>;
  __shared__ __attribute__((aligned(16))) float Wm[PPW][D * C::PITCH];
  const SolveArgs& p = a.tv.s;
  const int st = a.stride;
  const long long per = (p.T - st + 2LL * st - 1) / (2LL * st);  // elements j + st per problem in this round
  const long long items = p.n * per;
  const long long nquads = (items + PPW - 1) / PPW;
  for (long long quad = blockIdx.x; quad < nquads; quad += gridDim.x) {
    const int tid = threadIdx.x + opaque_zero(), lane = tid & 63, i = lane & 15, g = lane >> 4;
    constexpr int w = 0;
    float* const Wmine = Wm[g & (PPW - 1)];
    bool valid[PPW];
    float* out[PPW];  // the element's H in the workspace
    const float* e[PPW];
    const float* gP[PPW];
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
      valid[q] = quad * PPW + q < items;
      const long long item = valid[q] ? quad * PPW + q : items - 1;
      const long long prob = item / per;
      const long long j = (item % per) * 2 * st;
      // an element whose range reaches the terminal cost is a constant map: its H is P already, nothing to write; it
      // goes through the arithmetic on its own (finite) matrices with its own H standing in for the value on its right
      const bool reaches_end = j + 2 * st >= p.T;
      valid[q] = valid[q] && !reaches_end;
      e[q] = a.ws + (prob * p.T + j + st) * 3 * D * D;
      out[q] = a.ws + ((prob * p.T + j + st) * 3 + 2) * D * D;
      gP[q] = reaches_end ? e[q] + 2 * D * D : a.ws + ((prob * p.T + j + 2 * st) * 3 + 2) * D * D;
    }
    floatx4 accY[PPW][C::RB][C::NT], accR[PPW][C::RB][C::NT];
    float rAT[PPW][C::RB][C::KS];
    {
      float rP[PPW][C::RB][C::KS];
#pragma unroll
      for (int q = 0; q < PPW; ++q) {
        load_half<D, float, false>(Wm[q], e[q] + D * D, tid);  // G
        load_half<D, float, false>(Wm[q] + D, e[q], tid);      // A
        load_aop_global<D, float>(gP[q], rP[q], w, i, g);
        eye_acc<D>(accY[q], w, i, g);
        zero_acc<D>(accR[q]);
      }
      __syncthreads();
      gemm_acc_quad<PPW>(accY, rP, Wm, 0, i, g);  // I + P G
      gemm_acc_quad<PPW>(accR, rP, Wm, D, i, g);  // P A
#pragma unroll
      for (int q = 0; q < PPW; ++q) load_aopT_lds<D>(Wm[q] + D, rAT[q], w, i, g);
      __syncthreads();
#pragma unroll
      for (int q = 0; q < PPW; ++q) {
        store_rows<D>(Wm[q], accY[q], w, i, g);
        store_rows<D>(Wm[q] + D, accR[q], w, i, g);
      }
      __syncthreads();
    }
    const unsigned long long badm = __ballot(solve_rows16<true>(Wmine, lane) != 0);  // right halves: (I + P G)^{-1} P A
#pragma unroll
    for (int q = 0; q < PPW; ++q) load_rows_global<D>(e[q] + 2 * D * D, accY[q], w, i, g);
    gemm_acc_quad<PPW>(accY, rAT, Wm, D, i, g);
#pragma unroll
    for (int q = 0; q < PPW; ++q) {
      if ((badm >> (16 * q)) & 0xFFFFull) poison<D>(accY[q]);
      if (valid[q]) write_rows_global<D>(out[q], accY[q], w, i, g);
    }
    __syncthreads();
  }
}

}  // namespace ttc
