// ln_stats_kernel, gemm_ln_kernel, gemm_ln_bf16_kernel, gemm_ln_split_kernel, cxt_maps_kernel (ttc_block_forward).
#include "ttc_block.hpp"
#include "ttc_launch.hpp"

namespace ttc {
hipError_t launch_ln_stats(const LnStatsArgs& a, bool bf16, hipStream_t st) {
  const dim3 grid((unsigned)((a.M + 3) / 4 + a.r));
  if (bf16) hipLaunchKernelGGL((ln_stats_kernel<unsigned short>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((ln_stats_kernel<float>), grid, dim3(256), 0, st, a);
  return hipGetLastError();
}
static long long tiles_of(long long M, int N) {
  return ((M + GEMM_BM - 1) / GEMM_BM) * ((N + GEMM_BN - 1) / GEMM_BN);
}
// Which kernel forms a projection.  The tiled kernels (128 x 128 per workgroup) walk K one slice after the other with one
// slice in flight, whatever the number of tiles up to one per compute unit; below that number the kernel that shares K among
// a workgroup's wavefronts may be faster, with the largest tile that still gives every compute unit a workgroup, one to a
// compute unit at a time.  Measured in us, tiled / split, at N = 256 outputs, K = 4096:
// float32 M = 32 tokens 329 / 21, 512: 342 / 31, 2048: 344 / 61, 4096: 345 / 98, 8192 (128 tiles): 344 / 188; bfloat16
// M = 32: 92 / 14, 2048: 178 / 30, 8192: 177 / 74.  At N = 4096 a round of 64 x 64 tiles is 256 tokens: K = 256, float32
// M = 32: 25 / 6, 512 (two rounds): 30 / 22, 640: 31 / 32, 896 (four): 32 / 41; bfloat16 512: 15 / 14, 640: 16 / 20, 896: 16 / 26;
// K = 64, float32 384: 13 / 14, 640: 15 / 20; bfloat16 512: 10 / 9, 640: 10 / 12.  Both kernels' times are linear in K:
// tiled 8.5 us + 84 ns K (bfloat16 7.5 us + 40 ns K), a round of split 5.3 us + 20 ns K (3.9 us + 8 ns K).
static bool split_is_faster(long long M, int N, int K, int cus, bool bf16) {
  if (tiles_of(M, N) >= cus) return false;
  const long long tiles = ((M + 63) / 64) * ((N + 63) / 64), rounds = (tiles + cus - 1) / cus;
  const double split = (double)rounds * (bf16 ? 3900. + 8.2 * K : 5300. + 19.5 * K);
  return split <= 0.9 * (bf16 ? 7500. + 40. * K : 8500. + 84.4 * K);
}
// Whether the split kernel takes its smallest tile, 16 tokens by 16 outputs, whose sixteen wavefronts share K.
static bool smallest_tile(long long M, int N, int cus) { return ((N + 15) / 16) * ((M + 31) / 32) < cus; }
// Short rows are read so fast that the split kernel forms their statistics itself where it takes its smallest tile: a row to each of the
// workgroup's wavefronts, which costs less than a launch for them.  With larger tiles a wavefront forms those of four or eight rows one after
// the other, in every workgroup, which costs more.  The block with / without the launch, us a call, K = 256: 1024 outputs, 32 tokens 31.2 /
// 29.6, 128 37.6 / 38.7; 2048 outputs, 16 tokens 35.9 / 34.5, 32 36.5 / 35.0, 33 37.1 / 38.3; 4096 outputs, 32 tokens 47.5 / 48.8; K = 64,
// 4096 outputs, 150 tokens 51.6 / 56.3, 1024 outputs, 400 tokens 39.6 / 44.2.
bool stats_inside(long long M, int N, int K, int cus, bool bf16) {
  return K <= 512 && M * K <= 128 * 256 && smallest_tile(M, N, cus) && split_is_faster(M, N, K, cus, bf16);
}
template <typename TX, typename TW, typename TY>
static hipError_t launch_split(const GemmLnSplitArgs& a, int cus, hipStream_t st) {
  const long long n16 = (a.N + 15) / 16, n64 = (a.N + 63) / 64;
  const long long m16 = (a.M + 15) / 16, m32 = (a.M + 31) / 32, m64 = (a.M + 63) / 64;
  if (n64 * m64 >= cus)
    hipLaunchKernelGGL((gemm_ln_split_kernel<TX, TW, TY, 4, 4, 8>), dim3((unsigned)(n64 * m64)), dim3(512), 0, st, a);
  else if (n64 * m32 >= cus)
    hipLaunchKernelGGL((gemm_ln_split_kernel<TX, TW, TY, 4, 2, 8>), dim3((unsigned)(n64 * m32)), dim3(512), 0, st, a);
  else if (!smallest_tile(a.M, a.N, cus))
    hipLaunchKernelGGL((gemm_ln_split_kernel<TX, TW, TY, 1, 2, 8>), dim3((unsigned)(n16 * m32)), dim3(512), 0, st, a);
  else
    hipLaunchKernelGGL((gemm_ln_split_kernel<TX, TW, TY, 1, 1, 16>), dim3((unsigned)(n16 * m16)), dim3(1024), 0, st, a);
  return hipGetLastError();
}
// x_bf16: X is bfloat16 (else float32); out_bf16: Y is bfloat16 (else float32); exactly one of them (the two projections)
hipError_t launch_gemm_ln_bf16(const GemmLnBf16Args& a, bool x_bf16, bool out_bf16, int cus, hipStream_t st) {
  if (x_bf16 == out_bf16) return hipErrorInvalidValue;
  if (split_is_faster(a.M, a.N, a.K, cus, true)) {
    const GemmLnSplitArgs s{a.X, a.stats, a.gain, a.offset, a.W, a.bias, a.Res, a.Y, a.M, a.N, a.K, a.eps};
    if (x_bf16) return launch_split<unsigned short, unsigned short, float>(s, cus, st);
    return launch_split<float, unsigned short, unsigned short>(s, cus, st);
  }
  const dim3 grid((unsigned)(8 * ((tiles_of(a.M, a.N) + 7) / 8)));
  if (x_bf16) hipLaunchKernelGGL((gemm_ln_bf16_kernel<unsigned short, false>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((gemm_ln_bf16_kernel<float, true>), grid, dim3(256), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_gemm_ln(const GemmLnArgs& a, int cus, hipStream_t st) {
  if (split_is_faster(a.M, a.N, a.K, cus, false)) {
    const GemmLnSplitArgs s{a.X, a.stats, a.gain, a.offset, a.W, a.bias, a.Res, a.Y, a.M, a.N, a.K, a.eps};
    return launch_split<float, float, float>(s, cus, st);
  }
  hipLaunchKernelGGL(gemm_ln_kernel, dim3((unsigned)(8 * ((tiles_of(a.M, a.N) + 7) / 8))), dim3(256), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_cxt_maps(const CxtMapsArgs& a, int blocks, hipStream_t st) {
  if (a.r == 16 && a.H % 4 == 0) {  // `blocks` counts (token chunk, group of four heads) pairs here
    hipLaunchKernelGGL(cxt_maps16_kernel, dim3((unsigned)blocks), dim3(512), 0, st, a);
    return hipGetLastError();
  }
  const int nout = 80 + 3 * a.r;
  hipLaunchKernelGGL(cxt_maps_kernel, dim3((unsigned)blocks), dim3((unsigned)(64 * ((nout + 63) / 64))), 0, st, a);
  return hipGetLastError();
}
}  // namespace ttc
