// 2D stage in one launch with the corrections in place (gfx950, FP64).
//
// A workgroup takes a tile of 63 columns x R rows: its wavefronts load the
// tile's records with three halo cells a side into LDS, then each takes one
// row of faces (R rows of x faces, R + 1 rows of y faces: 2 R + 1 wavefronts)
// with their WENO corrections (wave_face), and after a barrier the cells are
// updated.  The chain of a stage is one load, one face, one correction and two
// barriers, where the row kernel marches through its rows and lists the
// flagged cells (an atomic per wavefront and row on one counter) for a second
// launch that loads their stencils again.  The price is more halo records and
// (R + 1) / R of the y faces, so large grids whose faces are mostly linear keep
// the row kernel (the rule is at use_tile).  The arithmetic is the row
// kernel's and its correction kernel's, operation for operation: the same
// bits.
#pragma once
#include "wl2_aux.hpp"
#include "wl2_row.hpp"
#include "wl2_wface.hpp"

namespace wl2 {

constexpr int TV = 4;           // conserved values in 2D
constexpr int TVP = RB + 1;     // doubles between two values of a record row
constexpr int TROW = (TV + 3) * TVP;  // doubles of a record row

struct TileArgs {
  RowArgs r;
  StepCtl* commit;     // stage 2: commit the clock that stage 1 formed (or null)
  int yghosts;         // the grid has y state sides (rule)
  YGhostRule rule;
  double dx, tc;       // cell size; time of this stage's ghosts (yghost_time)
};

template <int R>
struct TileShared {
  static constexpr int NW = 2 * R + 1;
  double rec[(R + 6) * TROW];
  double sF[NW][TV][64];         // first a wavefront's scratch, then its fluxes
  FaceScratch<TV> scr[NW];       // dv of a wavefront: later its dF
  unsigned long long smask[NW];  // flagged faces of a wavefront
};

// The tile of columns x0 .. and rows y0 ..; record row k (0 .. R + 5) holds
// grid row y0 - 3 + k; position c column x0 - 3 + c.  lead: this workgroup
// writes what one of the grid writes (clock, cleared slots).
template <int R, int OUT, int SPLIT, int HYB, int W>
__device__ __forceinline__ void tile2d_item(const TileArgs& ta, const KGrid& g, const KPhys& ph, int x0,
                                            int y0, bool lead, TileShared<R>& sh) {
  constexpr int NV = TV, NW = 2 * R + 1, ROWS = R + 6;
  const RowArgs& a = ta.r;
  double* rec = sh.rec;
  double (*sF)[NV][64] = sh.sF;
  FaceScratch<NV>* scr = sh.scr;
  unsigned long long* smask = sh.smask;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // scalar: so are its rows
  const int rows = min(R, g.n[1] - y0);

  // loads: record rows (64 columns x0 .. x0 + 63 each) and, last, the five
  // columns x0 - 3 .. x0 - 1, x0 + 64, x0 + 65 of the tile's own rows, dealt
  // to the wavefronts; all issued before the first use
  constexpr int LOADS = ROWS + 1, PER = (LOADS + NW - 1) / NW;
  double u[PER][NV];
  int pos[PER];
  bool neg1[PER], neg2[PER];  // mirror ghosts: the momenta to negate once loaded
  bool fxl = false;
  int cxl = x0 + lane;
  if (x0 + 63 >= g.n[0]) cxl = ghost_clamped(cxl, g.n[0], g.bc_lo[0], g.bc_hi[0], fxl);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int job = wave + i * NW;
    pos[i] = -1;
    neg1[i] = neg2[i] = false;
    int cx = cxl, iy = 0;
    if (job < rows + 6) {
      const int y = y0 - 3 + job;
      pos[i] = job * TROW + lane + 3;
      neg1[i] = fxl;
      iy = y;
      if (y < 0 || y >= g.n[1]) {
        if (ta.yghosts && is_yghost(g, y)) {
          yghost_value(a.Uk, g, yghost_time(a.ctl, ta.tc), ta.dx, ta.rule, cxl, y, u[i]);
          neg1[i] = false;
          iy = -1;  // formed, not loaded
        } else {
          iy = ghost_clamped(y, g.n[1], g.bc_lo[1], g.bc_hi[1], neg2[i]);
        }
      }
    } else if (job == ROWS && lane < 5 * rows) {
      const int row = 3 + lane / 5, q = lane % 5;
      const int x = x0 + (q < 3 ? q - 3 : 61 + q);
      iy = y0 - 3 + row;
      pos[i] = row * TROW + (x - x0 + 3);
      cx = ghost_clamped(x, g.n[0], g.bc_lo[0], g.bc_hi[0], neg1[i]);
      if (x < 0 && g.bc_lo[0] == BC_INFLOW) {
        load_inflow<NV>(g, iy, u[i]);
        iy = -1;
      }
    }
    if (pos[i] >= 0 && iy >= 0) {
      const long long o = cx + (long long)iy * g.stride[1];
#pragma unroll
      for (int v = 0; v < NV; ++v) u[i][v] = a.Uk[v * g.ncell + o];
    }
  }
  // global LF speeds along this wavefront's faces
  unsigned long long lf[NV] = {};
  if (SPLIT == SPLIT_LF || (SPLIT < 0 && ph.split == SPLIT_LF)) {
    const int d = wave < R ? 0 : 1;
    if (a.lf_in != nullptr) {
      lf_take_wave<NV>(a.lf_in, d, lf);
    } else {
#pragma unroll
      for (int k = 0; k < NV; ++k) lf[k] = a.ctl->lf_bits[d][k];
    }
    if (a.lf_clear != nullptr && lead && threadIdx.x < LF_SLOTS) a.lf_clear[threadIdx.x] = LfSlot{};
  }
  // U^n of the cell this lane updates
  const int uy = y0 + wave;
  const bool own = wave < rows && lane < RT && x0 + lane < g.n[0];
  const long long off = (long long)(x0 + lane) + (long long)uy * g.stride[1];
  double unp[NV] = {};
  if (OUT == OUT_RK && a.rk_a != 0.0 && own) {
#pragma unroll
    for (int v = 0; v < NV; ++v) unp[v] = __builtin_nontemporal_load(&a.Un[v * g.ncell + off]);
  }
  double dt = 0.0;
  if (OUT == OUT_RK) {
    dt = a.clock != nullptr
             ? clock_dt_wave(a.clock, a.cfl_dx, a.s_floor, lead && threadIdx.x == 0)
             : a.ctl->dt;
    // (a stopped step's clock too: the CFL maximum that it found must not meet
    // the next reduction's)
    if (ta.commit != nullptr && lead && threadIdx.x == 0) clock_commit(ta.commit);
    if (!(dt > 0.0)) return;  // finished run: leave the state untouched (uniform)
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (pos[i] >= 0) {
      if (neg1[i]) u[i][1] = -u[i][1];
      if (neg2[i]) u[i][2] = -u[i][2];
      LRec<NV> r;
      make_lrec<NV>(u[i], ph, r);
      lane_put<NV, TVP>(rec + pos[i], r);
    }
  }
  __syncthreads();

  // faces: wavefront w < R the x faces left of the columns of row w, the
  // others the y faces below row w - R
  {
    double F60[NV], dF[NV];
    bool m = false;
    const bool live = wave < R ? wave < rows : wave - R <= rows;
    if (live) {
      if (wave < R)
        m = wave_face<NV, 0, TVP, SPLIT, HYB, W>(rec + (wave + 3) * TROW, 1, x0 + lane <= g.n[0], ph, lf,
                                                 scr[wave], sF[wave], F60, dF);
      else
        m = wave_face<NV, 1, TVP, SPLIT, HYB, W>(rec + (wave - R) * TROW + 3, TROW,
                                                 lane < RT && x0 + lane < g.n[0], ph, lf, scr[wave], sF[wave],
                                                 F60, dF);
#pragma unroll
      for (int v = 0; v < NV; ++v) sF[wave][v][lane] = F60[v];
      const unsigned long long mw = __ballot(m);
      if (lane == 0) smask[wave] = mw;
      if (m) {
#pragma unroll
        for (int v = 0; v < NV; ++v) scr[wave].dv[v][lane] = dF[v];
      }
    }
  }
  __syncthreads();

  double cfl_max = 0.0, mx[NV - 2][3] = {};
  bool cfl_bad = false;
  if (own) {
    const int jx = wave, jl = R + wave, jh = R + wave + 1;  // x, y-, y+ face rows
    const unsigned cm = (unsigned)((smask[jx] >> lane) & 3ull) | ((smask[jl] >> lane) & 1ull ? 4u : 0u) |
                        ((smask[jh] >> lane) & 1ull ? 8u : 0u);
    double acc[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = 0.0;
    if (cm) {
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        if (!((cm >> f) & 1u)) continue;
        const double sg = (f & 1) ? -1.0 : 1.0;
        const int j = f < 2 ? jx : (f == 2 ? jl : jh), l = f == 1 ? lane + 1 : lane;
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v] += sg * scr[j].dv[v][l];
      }
    }
    const double* ru = rec + (wave + 3) * TROW + lane + 3;
    const double scale = OUT == OUT_RK ? a.rk_b * dt : 1.0;
    double un[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const double dU = ((sF[jx][v][lane] - sF[jx][v][lane + 1]) + (sF[jl][v][lane] - sF[jh][v][lane])) * ph.inv_dx60;
      double r = dU;
      if (OUT == OUT_RK) {
        r = a.rk_b * (ru[v * TVP] + dt * dU);
        if (a.rk_a != 0.0) r += a.rk_a * unp[v];
      }
      if (cm) r = r + scale * (acc[v] * ph.inv_dx);
      __builtin_nontemporal_store(r, &a.out[v * g.ncell + off]);
      un[v] = r;
    }
    if (OUT == OUT_RK && a.cfl != nullptr) cfl_max = nan_max(cfl_max, cfl_speed_u<NV>(un, ph.gamma, cfl_bad));
    if (OUT == OUT_RK && a.lf_out != nullptr) lf_fold_cell<NV>(un, ph.gamma, mx);
  }
  if (OUT == OUT_RK && wave < rows) {
    if (a.lf_out != nullptr) lf_commit_wave<NV - 2>(a.lf_out, mx);
    if (a.cfl != nullptr) cfl_commit_wave(a.cfl, cfl_max, cfl_bad);
  }
}

// Tiles first + blockIdx.x (unsigned: a signed division costs each wavefront's
// start 0.2 us).
template <int R, int OUT, int SPLIT, int HYB, int W>
__global__ __launch_bounds__((2 * R + 1) * 64, 4) void tile2d_kernel(TileArgs ta, KGrid g, KPhys ph,
                                                                    unsigned tiles_x, unsigned first) {
  __shared__ TileShared<R> sh;
  const unsigned b = first + blockIdx.x;
  tile2d_item<R, OUT, SPLIT, HYB, W>(ta, g, ph, (int)(b % tiles_x) * RT, (int)(b / tiles_x) * R, b == 0u, sh);
}

}  // namespace wl2
