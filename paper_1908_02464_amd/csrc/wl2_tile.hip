// Dispatch of the 2D tile kernels (wl2_tile.hpp).
#include <hip/hip_runtime.h>

#include "wl2_row_launch.hpp"
#include "wl2_tile.hpp"

namespace wl2 {

hipError_t tile2d_launch(const RowLaunch& L, int rows) {
  if (L.nvar != 4) return hipErrorInvalidValue;
  TileArgs ta{};
  RowArgs& a = ta.r;
  a.Uk = L.Uk;
  a.out = L.out;
  a.Un = L.Un;
  a.ctl = L.ctl;
  a.rk_a = L.rk_a;
  a.rk_b = L.rk_b;
  if (L.out_kind == OUT_RK) {
    a.cfl = L.cfl;
    a.clock = L.clock;
    ta.commit = L.commit;
    a.lf_in = L.lf_in;
    a.lf_out = L.lf_out;
    a.lf_clear = L.lf_clear;
  }
  a.cfl_dx = L.cfl_dx;
  a.s_floor = L.s_floor;
  ta.yghosts = L.rule != nullptr;
  if (L.rule != nullptr) ta.rule = *L.rule;
  ta.dx = L.dx;
  ta.tc = L.tc;
  const unsigned tiles_x = (unsigned)((L.g.n[0] + RT - 1) / RT);
  const long long blocks = (long long)tiles_x * ((L.g.n[1] + rows - 1) / rows);
  if (blocks < 1 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  // a launch holds at most 2^32 - 1 lanes (9.6 M tiles): more go in several
  // (their order does not matter: only tile 0 writes what the others read in
  // a later stage)
  const int most = (int)(0xffffffffLL / ((2 * rows + 1) * 64));
  const bool w0 = L.ph.weights == W_L2IS;
  // builds: the per-field switch with LLF or global LF splitting and the
  // weights of Eq.(28) fixed at compile time, any other scheme read at run time
#define WL2_TILE_BUILD(R, O, S, H, W) \
  hipLaunchKernelGGL((tile2d_kernel<R, O, S, H, W>), gr, dim3((2 * R + 1) * 64), 0, L.stream, ta, L.g, L.ph, tiles_x, first)
#define WL2_TILE(R, O)                                                              \
  do {                                                                              \
    if (w0 && L.fast == 1) WL2_TILE_BUILD(R, O, SPLIT_LLF, HYB_PER_FIELD, W_L2IS);     \
    else if (w0 && L.fast == 2) WL2_TILE_BUILD(R, O, SPLIT_LF, HYB_PER_FIELD, W_L2IS); \
    else WL2_TILE_BUILD(R, O, -1, -1, -1);                                          \
  } while (0)
#define WL2_TILE_OUT(R)                                \
  do {                                                 \
    if (L.out_kind == OUT_RK) WL2_TILE(R, OUT_RK);     \
    else WL2_TILE(R, OUT_WRITE);                       \
  } while (0)
  if (rows != 1 && rows != 3) return hipErrorInvalidValue;
  hipError_t e = hipSuccess;
  for (long long f = 0; f < blocks && e == hipSuccess; f += most) {
    const unsigned first = (unsigned)f;
    const dim3 gr((unsigned)(blocks - f < most ? blocks - f : most));
    if (rows == 1) WL2_TILE_OUT(1);
    else WL2_TILE_OUT(3);
    e = hipGetLastError();
  }
  return e;
#undef WL2_TILE_OUT
#undef WL2_TILE
#undef WL2_TILE_BUILD
}

}  // namespace wl2
