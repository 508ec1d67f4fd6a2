// Dispatch of the 1D whole-step kernels (wl2_line.hpp).
#include <hip/hip_runtime.h>

#include "wl2_line.hpp"

namespace wl2 {

static_assert(LINE_STEPS_MAX_CELLS == 8 * LW, "eight wavefronts");
static_assert(sizeof(LineCtl) == LINE_CTL_BYTES, "size known to the context");

// Builds: the default scheme (LLF splitting, per-field switch, Eq.(28)) fixed
// at compile time, any other read at run time.
static bool line_default(const KPhys& ph) {
  return ph.split == SPLIT_LLF && ph.hybrid == HYB_PER_FIELD && ph.weights == W_L2IS;
}

hipError_t line_steps(double* U, StepCtl* ctl, double cfl_dx, int n_steps, const KGrid& g, const KPhys& ph,
                      hipStream_t stream) {
  if (g.n[1] != 1 || g.n[2] != 1 || g.n[0] > LINE_STEPS_MAX_CELLS) return hipErrorInvalidValue;
  const LineStepsArgs s{U, ctl, cfl_dx, n_steps};
#define WL2_LS(NW)                                                                                  \
  do {                                                                                              \
    if (line_default(ph))                                                                           \
      hipLaunchKernelGGL((line_steps_kernel<NW, SPLIT_LLF, HYB_PER_FIELD, W_L2IS>), dim3(1),    \
                         dim3(NW * 64), 0, stream, s, g, ph);                                       \
    else                                                                                            \
      hipLaunchKernelGGL((line_steps_kernel<NW, -1, -1, -1>), dim3(1), dim3(NW * 64), 0, stream, \
                         s, g, ph);                                                                 \
  } while (0)
  // one wavefront per SIMD where the cells allow it (shock / entropy wave: 252
  // cells on four wavefronts 8.7 us per step, 253 on eight 11.9)
  if (g.n[0] <= 4 * LW) WL2_LS(4);
  else WL2_LS(8);
#undef WL2_LS
  return hipGetLastError();
}

hipError_t line_advance(double* U, double* tmp, LineCtl* lc, StepCtl* ctl, double cfl_dx, double s_floor,
                        int n_steps, double t_end, const KGrid& g, const KPhys& ph, hipStream_t stream) {
  const int n = g.n[0];
  if (g.n[1] != 1 || g.n[2] != 1 || n > LINE_MAX_CELLS) return hipErrorInvalidValue;
  hipLaunchKernelGGL(line_begin_kernel, dim3(1), dim3(64), 0, stream, lc, ctl, t_end);
  if (n_steps < 1) return hipGetLastError();
  const int rb = (n + RED_BLOCK - 1) / RED_BLOCK;
  hipLaunchKernelGGL(line_cfl_kernel, dim3(rb < 1024 ? rb : 1024), dim3(RED_BLOCK), 0, stream, U, n, ph.gamma,
                     lc, (n_steps & 1) ? tmp : nullptr);
  const dim3 gr((n + LT - 1) / LT), bl(64);
  for (int i = 0; i < n_steps; ++i) {
    const bool to_u = ((n_steps - i) & 1) != 0;  // the last step writes U
    const LineStepArgs a{to_u ? tmp : U, to_u ? U : tmp, lc, ctl, cfl_dx, s_floor, i, i + 1 < n_steps};
    if (line_default(ph))
      hipLaunchKernelGGL((line_step_kernel<SPLIT_LLF, HYB_PER_FIELD, W_L2IS>), gr, bl, 0, stream, a, g, ph);
    else
      hipLaunchKernelGGL((line_step_kernel<-1, -1, -1>), gr, bl, 0, stream, a, g, ph);
  }
  hipLaunchKernelGGL(line_end_kernel, dim3(1), dim3(64), 0, stream, lc, ctl, n_steps);
  return hipGetLastError();
}

}  // namespace wl2
