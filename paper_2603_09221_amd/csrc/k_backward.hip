// The kernels of ttc_lqr_backward, ttc_lqr_backward_tv: one translation unit per state size (d = 16: backward16_kernel, one
// wavefront per problem; backward_kernel<TTC_D> otherwise).
#if TTC_D == 16
#include "ttc_backward16.hpp"
#else
#include "ttc_backward.hpp"
#endif
#include "ttc_launch.hpp"

namespace ttc {
#if TTC_D == 16
template <typename TIn>
static constexpr auto kernel = backward16_kernel<TIn, false>;
#else
template <typename TIn>
static constexpr auto kernel = backward_kernel<TTC_D, TIn>;
#endif
template <>
hipError_t launch_backward<TTC_D>(const BackwardArgs& a, bool bf16, dim3 grid, hipStream_t st) {
#if TTC_D == 16
  if (a.past_caches) {
    if (bf16) hipLaunchKernelGGL((backward16_kernel<uint16_t, true>), grid, dim3(64), 0, st, a);
    else hipLaunchKernelGGL((backward16_kernel<float, true>), grid, dim3(64), 0, st, a);
    return hipGetLastError();
  }
#endif
  if (bf16) hipLaunchKernelGGL(kernel<uint16_t>, grid, dim3(Cfg<TTC_D>::NTHR), 0, st, a);
  else hipLaunchKernelGGL(kernel<float>, grid, dim3(Cfg<TTC_D>::NTHR), 0, st, a);
  return hipGetLastError();
}
template <>
int occupancy_backward<TTC_D>(bool bf16) {
  return bf16 ? occupancy_query(kernel<uint16_t>, Cfg<TTC_D>::NTHR) : occupancy_query(kernel<float>, Cfg<TTC_D>::NTHR);
}
}  // namespace ttc
