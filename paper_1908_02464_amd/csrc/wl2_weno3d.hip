// Dispatch of the 3D stage with every face WENO (wl2_weno3d.hpp).
#include <hip/hip_runtime.h>

#include "wl2_weno3d.hpp"

namespace wl2 {

namespace {

// Cells that a lane marches through: the tuned value, else the balanced one; at
// least as many as keep a launch of `groups` wavefronts per chunk within the
// runtime's 2^32 - 1 lanes.
int march(const FusedLaunch& L, long long groups, int n) {
  const int len = L.march > 0 ? L.march : balanced_chunk(groups, n, 1, 64);
  const long long chunks = (0xffffffffLL / 64) / groups;
  const long long least = chunks > 0 ? (n + chunks - 1) / chunks : n;
  return len > least ? len : (int)least;
}

template <int OUT, int SPLIT, int W>
hipError_t launch(const FusedLaunch& L) {
  const Weno3dArgs a{L.Uk,   L.out,        L.Un, L.ctl, L.rk_a,
                     L.rk_b, L.list_clear, L.out_kind == OUT_RK ? L.cfl : nullptr, L.fo3};
  const long long nx = L.n[0], ny = L.n[1], nz = L.n[2];
  const long long bx = ((nx + 1) * ny * nz + WX_FACES - 1) / WX_FACES;
  const long long gy = (nx * nz + 63) / 64, gz = (nx * ny + 63) / 64;
  const int ly = march(L, gy, L.n[1]), lz = march(L, gz, L.n[2]);
  const long long by = gy * ((ny + ly - 1) / ly), bz = gz * ((nz + lz - 1) / lz);
  if (bx > 0x7fffffffLL || by > 0x7fffffffLL || bz > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 b(64);
  hipLaunchKernelGGL((weno3d_x_kernel<OUT, SPLIT, W>), dim3((unsigned)bx), b, 0, L.stream, a, L.g, L.ph);
  hipLaunchKernelGGL((weno3d_march_kernel<OUT, 1, SPLIT, W>), dim3((unsigned)by), b, 0, L.stream, a, L.g, L.ph, ly,
                     (unsigned)gy);
  hipLaunchKernelGGL((weno3d_march_kernel<OUT, 2, SPLIT, W>), dim3((unsigned)bz), b, 0, L.stream, a, L.g, L.ph, lz,
                     (unsigned)gz);
  return hipGetLastError();
}

template <int OUT, int SPLIT>
hipError_t launch_weights(const FusedLaunch& L) {
  switch (L.ph.weights) {
    case W_L2IS: return launch<OUT, SPLIT, W_L2IS>(L);
    case W_IS: return launch<OUT, SPLIT, W_IS>(L);
    default: return launch<OUT, SPLIT, W_IS_B01>(L);
  }
}

}  // namespace

// One build per weighting: a choice at run time keeps the values of all three
// in registers (392 of them, one wave per SIMD).  LLF splitting (the paper's)
// fixed at compile time, any other read at run time.
hipError_t weno3d_stage(const FusedLaunch& L) {
  const bool rk = L.out_kind == OUT_RK;
  if (L.ph.split == SPLIT_LLF)
    return rk ? launch_weights<OUT_RK, SPLIT_LLF>(L) : launch_weights<OUT_WRITE, SPLIT_LLF>(L);
  return rk ? launch_weights<OUT_RK, -1>(L) : launch_weights<OUT_WRITE, -1>(L);
}

}  // namespace wl2
