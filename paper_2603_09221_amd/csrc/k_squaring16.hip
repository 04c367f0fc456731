// squaring16_kernel (ttc_lqr_solve at d = 16, default path): one or four problems per wavefront.
#include "ttc_squaring16.hpp"
#include "ttc_launch.hpp"

namespace ttc {
template <typename TIn, int PPW>
static void launch(const DoublingArgs& a, dim3 grid, hipStream_t st) {
  if (a.p_from_qt) hipLaunchKernelGGL((squaring16_kernel<TIn, PPW, true>), grid, dim3(64), 0, st, a);
  else hipLaunchKernelGGL((squaring16_kernel<TIn, PPW, false>), grid, dim3(64), 0, st, a);
}
hipError_t launch_squaring16(const DoublingArgs& a, bool bf16, int ppw, dim3 grid, hipStream_t st) {
  if (ppw == 4) {
    if (bf16) launch<uint16_t, 4>(a, grid, st);
    else launch<float, 4>(a, grid, st);
  } else {
    if (bf16) launch<uint16_t, 1>(a, grid, st);
    else launch<float, 1>(a, grid, st);
  }
  return hipGetLastError();
}
int occupancy_squaring16(bool bf16, int ppw) {
  if (ppw == 1)
    return bf16 ? occupancy_query(squaring16_kernel<uint16_t, 1, false>, 64) : occupancy_query(squaring16_kernel<float, 1, false>, 64);
  return bf16 ? occupancy_query(squaring16_kernel<uint16_t, 4, false>, 64) : occupancy_query(squaring16_kernel<float, 4, false>, 64);
}
}  // namespace ttc
