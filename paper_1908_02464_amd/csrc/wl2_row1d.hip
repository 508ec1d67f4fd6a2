// Corrections of long 1D lists (row_fix_kernel at three wavefronts per SIMD).
// A code object of their own: beside the row kernels they shifted those within
// theirs, which moved the times of 2D steps by up to 1 % either way.
#include <hip/hip_runtime.h>

#include "wl2_row.hpp"
#include "wl2_row_launch.hpp"

namespace wl2 {

hipError_t row_fix_three_waves(const RowLaunch& L, const RowArgs& a, dim3 grid, dim3 block) {
  if (L.out_kind == OUT_RK)
    hipLaunchKernelGGL((row_fix_kernel<3, OUT_RK, -1, -1, 3>), grid, block, 0, L.stream, a, L.g, L.ph);
  else
    hipLaunchKernelGGL((row_fix_kernel<3, OUT_WRITE, -1, -1, 3>), grid, block, 0, L.stream, a, L.g, L.ph);
  return hipGetLastError();
}

}  // namespace wl2
