// Dispatch of the fused 1D/2D row kernels (wl2_row.hpp).
#include <hip/hip_runtime.h>

#include "wl2_row.hpp"
#include "wl2_row_launch.hpp"

namespace wl2 {

static_assert(ROW_TILE == RT, "one tile width for host and device");

namespace {

// Builds: the splitting and the switch fixed at compile time (per field and per
// face ask the same question here: whether any field needs the nonlinear flux).
// Read at run time, they spill 50 to 90 registers: 6 to 14 % slower at 1100x900.
template <int NV, int OUT, int SPLIT>
void launch_split(const RowLaunch& L, const RowArgs& a, dim3 grid, int ych, int tiles_x) {
#define WL2_ROW(H) \
  hipLaunchKernelGGL((row_kernel<NV, OUT, SPLIT, H>), grid, dim3(RW), 0, L.stream, a, L.g, L.ph, ych, tiles_x)
  if (L.ph.hybrid == HYB_WENO_ONLY) WL2_ROW(HYB_WENO_ONLY);
  else if (L.ph.hybrid == HYB_LINEAR_ONLY) WL2_ROW(HYB_LINEAR_ONLY);
  else WL2_ROW(HYB_PER_FIELD);
#undef WL2_ROW
}

template <int NV, int OUT>
void launch_nv(const RowLaunch& L, const RowArgs& a, dim3 grid, int ych, int tiles_x) {
  if (L.ph.split == SPLIT_LLF) launch_split<NV, OUT, SPLIT_LLF>(L, a, grid, ych, tiles_x);
  else if (L.ph.split == SPLIT_LF) launch_split<NV, OUT, SPLIT_LF>(L, a, grid, ych, tiles_x);
  else launch_split<NV, OUT, SPLIT_ROE>(L, a, grid, ych, tiles_x);
}

}  // namespace

hipError_t row_reset(const RowLaunch& L) {
  hipLaunchKernelGGL(row_list_reset_kernel, dim3(1), dim3(64), 0, L.stream, L.list_n);
  if (L.list_clear != nullptr)
    hipLaunchKernelGGL(row_list_reset_kernel, dim3(1), dim3(64), 0, L.stream, L.list_clear);
  return hipGetLastError();
}

hipError_t row_fix(const RowLaunch& L) {
  const RowArgs a{L.Uk,   L.out,    L.Un, L.ctl,        L.rk_a,
                  L.rk_b, L.list,   L.list_n, L.list_clear,
                  L.out_kind == OUT_RK ? L.cfl : nullptr, L.out_kind == OUT_RK ? L.clock : nullptr,
                  L.cfl_dx, L.s_floor, L.lf_in, L.lf_out, L.lf_clear};
  const dim3 fg(1024), fb(128);
  // the per-cell kernel: 2048 workgroups, so that lists of up to 16384
  // cells take its field-parallel mode (workgroups past the list's end
  // return at once)
  const dim3 fgc(2048);
  if (L.fo_D != nullptr) {
    if (L.nvar != 4) return hipErrorInvalidValue;
#define WL2_FO(O, S, H)                                                                          \
  do {                                                                                           \
    hipLaunchKernelGGL((row_face_kernel<4, O, S, H>), fg, fb, 0, L.stream, a, L.g, L.ph, L.fo_D,  \
                       L.fo_map, L.fo_cap);                                                      \
    hipLaunchKernelGGL((row_sum_kernel<4, O, S, H>), fg, fb, 0, L.stream, a, L.g, L.ph, L.fo_D,   \
                       L.fo_map, L.fo_cap);                                                      \
  } while (0)
    if (L.out_kind == OUT_RK) {
      if (L.fast == 1) WL2_FO(OUT_RK, SPLIT_LLF, HYB_PER_FIELD);
      else if (L.fast == 2) WL2_FO(OUT_RK, SPLIT_LF, HYB_PER_FIELD);
      else WL2_FO(OUT_RK, -1, -1);
    } else {
      if (L.fast == 1) WL2_FO(OUT_WRITE, SPLIT_LLF, HYB_PER_FIELD);
      else if (L.fast == 2) WL2_FO(OUT_WRITE, SPLIT_LF, HYB_PER_FIELD);
      else WL2_FO(OUT_WRITE, -1, -1);
    }
#undef WL2_FO
    return hipGetLastError();
  }
  // two wavefronts per SIMD hold 131072 cells
  if (L.nvar == 3 && L.fast == 0 && L.g.ncell > 131072) return row_fix_three_waves(L, a, fgc, fb);
#define WL2_FIX_BUILD(NV, O, S, H) \
  hipLaunchKernelGGL((row_fix_kernel<NV, O, S, H, 2>), fgc, fb, 0, L.stream, a, L.g, L.ph)
#define WL2_FIX(NV, O)                                                \
  do {                                                                \
    if (L.fast == 1) WL2_FIX_BUILD(NV, O, SPLIT_LLF, HYB_PER_FIELD);     \
    else if (L.fast == 2) WL2_FIX_BUILD(NV, O, SPLIT_LF, HYB_PER_FIELD); \
    else WL2_FIX_BUILD(NV, O, -1, -1);                                \
  } while (0)
  if (L.nvar == 3) {
    if (L.out_kind == OUT_RK) WL2_FIX(3, OUT_RK); else WL2_FIX(3, OUT_WRITE);
  } else if (L.nvar == 4) {
    if (L.out_kind == OUT_RK) WL2_FIX(4, OUT_RK); else WL2_FIX(4, OUT_WRITE);
  } else {
    return hipErrorInvalidValue;
  }
#undef WL2_FIX_BUILD
#undef WL2_FIX
  return hipGetLastError();
}

hipError_t row_launch(const RowLaunch& L) {
  const RowArgs a{L.Uk,   L.out,  L.Un,     L.ctl, L.rk_a,
                  L.rk_b, L.list, L.list_n, nullptr,
                  L.out_kind == OUT_RK ? L.cfl : nullptr, L.out_kind == OUT_RK ? L.clock : nullptr,
                  L.cfl_dx, L.s_floor, L.lf_in, L.lf_out, L.lf_clear};
  if (L.nvar == 4 && L.g.n[0] > ROW_MAX_NX) return hipErrorInvalidValue;
  const int tiles_x = (L.g.n[0] + RT - 1) / RT;
  const int ych = L.nvar == 3 ? 1 : (L.ych < 1 ? 1 : (L.ych > ROW_MAX_YCH ? ROW_MAX_YCH : L.ych));
  const long long chunks = L.nvar == 3 ? 1 : (L.g.n[1] + ych - 1) / ych;
  const long long items = (long long)tiles_x * chunks;
  if (items < 1 || items > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 grid((unsigned)items);
  if (L.nvar == 3) {
    if (L.out_kind == OUT_RK) launch_nv<3, OUT_RK>(L, a, grid, ych, tiles_x);
    else launch_nv<3, OUT_WRITE>(L, a, grid, ych, tiles_x);
  } else if (L.nvar == 4) {
    if (L.out_kind == OUT_RK) launch_nv<4, OUT_RK>(L, a, grid, ych, tiles_x);
    else launch_nv<4, OUT_WRITE>(L, a, grid, ych, tiles_x);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace wl2
