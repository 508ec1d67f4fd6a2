// Launch interface of the fused 1D/2D row kernels (wl2_row.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "wl2_device.hpp"

namespace wl2 {

constexpr int ROW_TILE = 63;     // columns per work item (one wavefront)
constexpr int ROW_MAX_YCH = 62;  // rows per work item (the range that tune() states)
constexpr int ROW_MAX_NX = 1 << 29;  // columns of a 2D grid: a 32-bit byte offset

struct YGhostRule;

struct RowLaunch {
  const double* Uk;
  double* out;
  const double* Un;
  StepCtl* ctl;
  double rk_a, rk_b;
  int out_kind;  // OUT_WRITE or OUT_RK
  int ych;       // rows per work item (2D)
  int fast;      // compile-time build with the per-field switch: 1 = LLF
                 // splitting, 2 = global LF splitting, 0 = the scheme read at
                 // run time
  int nvar;      // 3 (1D) or 4 (2D)
  unsigned long long* list;  // correction list (ncell entries) and its length
  unsigned int* list_n;
  unsigned int* list_clear;  // the next stage's counter, zeroed by the correction kernel
  StepCtl* cfl;              // RK: fold the CFL speed of the new state here (or null)
  StepCtl* clock;            // RK stage 1: the stage kernel forms the step's dt
                             // from the CFL maximum folded here (or null)
  double cfl_dx, s_floor;    // with clock: CFL number x dx, inflow speed floor
  const LfSlot* lf_in;       // LF splitting: speeds of the input (null: ctl->lf_bits),
  LfSlot* lf_out;            // where the output's are folded (or null),
  LfSlot* lf_clear;          // and the set to clear for the next stage (or null)
  // tile kernel only
  StepCtl* commit;           // stage 2: commit the clock that stage 1 formed (or null)
  const YGhostRule* rule;    // state ghosts of the y sides (or null: none)
  double dx, tc;             // with them: cell size and stage time (yghost_time)
  // face-once corrections (2D, long lists): per-entry face changes
  // [2][nvar][fo_cap] and the cell -> entry map [ncell]; null: per cell
  double* fo_D;
  unsigned int* fo_map;
  unsigned int fo_cap;
  KGrid g;
  KPhys ph;
  hipStream_t stream;
};

// The launches of one stage, in stream order: the row kernel and the
// nonlinear corrections of the listed cells (2D grids up to ROW_MAX_NX wide).
// The list counter of a stage is
// cleared by the previous stage's correction kernel; row_reset clears both
// counters (before the first stage, or after a failed launch).
hipError_t row_reset(const RowLaunch& L);
hipError_t row_launch(const RowLaunch& L);
hipError_t row_fix(const RowLaunch& L);
// row_fix of a 1D list whose scheme is read at run time, three wavefronts per SIMD.
struct RowArgs;
hipError_t row_fix_three_waves(const RowLaunch& L, const RowArgs& a, dim3 grid, dim3 block);

// 2D: one stage with its corrections in one launch, `rows` (1 or 3) rows per
// workgroup (list and face-once members unused).
hipError_t tile2d_launch(const RowLaunch& L, int rows);

// 1D grids: n_steps clock steps of U (SSP-RK3, device CFL dt, the clock rule
// of finalize_dt_kernel; not with global LF splitting, whose speeds need a
// grid-wide reduction per stage).  line_steps: up to 504 cells, one
// single-workgroup launch for all steps (no inflow side).  line_advance: up to
// LINE_MAX_CELLS, one launch per step; tmp: a second state array.
constexpr int LINE_STEPS_MAX_CELLS = 504;
constexpr int LINE_MAX_CELLS = 0x7fffffff - (1 << 20);  // their 32-bit positions run on past the last cell
constexpr size_t LINE_CTL_BYTES = 3 * CFL_SLOTS * 128 + 128;
struct LineCtl;
hipError_t line_steps(double* U, StepCtl* ctl, double cfl_dx, int n_steps, const KGrid& g, const KPhys& ph,
                      hipStream_t stream);
hipError_t line_advance(double* U, double* tmp, LineCtl* lc, StepCtl* ctl, double cfl_dx, double s_floor,
                        int n_steps, double t_end, const KGrid& g, const KPhys& ph, hipStream_t stream);

}  // namespace wl2
