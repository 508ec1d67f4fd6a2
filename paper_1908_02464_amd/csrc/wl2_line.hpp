// Whole SSP-RK3 steps of a 1D grid in one launch (gfx950, FP64).
//
// A 1D grid is small: a stage of 1600 cells is under a microsecond of work, so
// launches and memory round trips, not the arithmetic, set its time (a stage
// kernel and a correction kernel per stage took 10.6 us at 1600 cells).  The
// state's three stages therefore stay on the chip:
//  * line_steps_kernel: the whole grid (up to 504 cells) in one workgroup,
//    which runs every step of the call, its records in LDS;
//  * line_step_kernel: larger grids, one launch per step (measured at 505 to
//    1008 cells: 10 us per step against 11 to 14 for one workgroup with two
//    cells per lane; at 400 cells one workgroup takes 8.0).  A wavefront loads
//    LT = 46 cells with nine halo cells on both sides and computes the three
//    stages on a range that shrinks by three cells per side and stage; only
//    the first and the last state touch memory.  The halo cells are computed
//    by both neighbours from the same values, so with the same bits.
// A flagged face is corrected where it is found (wave_face).  The arithmetic of
// a face, of its correction and of a cell's update is that of the stage kernels
// (row_item, row_fix_kernel), operation for operation: the same bits.
// Measured, us per step (before: stage and correction launches, and up to
// 1024 cells one workgroup through global memory): Riemann problem 200 cells
// 16.5 -> 7.7, shock / entropy wave 1600 cells 32 -> 10, every face WENO 8192
// cells 40 -> 17 and 400000 cells 360 -> 86.
#pragma once
#include "wl2_aux.hpp"
#include "wl2_row_launch.hpp"
#include "wl2_wface.hpp"

namespace wl2 {

constexpr int LNV = 3;
constexpr int LW = 63;  // cells of a wavefront's 64 faces

// Stage update of one cell from its two faces (row_item's and
// row_fix_kernel's operations): u becomes the stage's result.
__device__ __forceinline__ void line_update(double (&u)[LNV], const double (&un)[LNV], const double (&Fl)[LNV],
                                            const double (&Fr)[LNV], bool ml, bool mr,
                                            const double (&dl)[LNV], const double (&dr)[LNV], double rk_a,
                                            double rk_b, double dt, const KPhys& ph) {
  const double scale = rk_b * dt;
#pragma unroll
  for (int v = 0; v < LNV; ++v) {
    const double dU = (Fl[v] - Fr[v]) * ph.inv_dx60;
    double r = rk_b * (u[v] + dt * dU);
    if (rk_a != 0.0) r += rk_a * un[v];
    if (ml || mr) {
      double acc = 0.0;
      if (ml) acc += 1.0 * dl[v];
      if (mr) acc += -1.0 * dr[v];
      r = r + scale * (acc * ph.inv_dx);
    }
    u[v] = r;
  }
}

__device__ __forceinline__ void line_rk(int st, double& rk_a, double& rk_b) {
  rk_a = st == 0 ? 0.0 : (st == 1 ? 0.75 : 1.0 / 3.0);
  rk_b = st == 0 ? 1.0 : (st == 1 ? 0.25 : 2.0 / 3.0);
}

struct LineStepsArgs {
  double* U;      // state, advanced in place
  StepCtl* ctl;   // clock, t_end, status, dt
  double cfl_dx;  // CFL number x dx
  int n_steps;
};

// Every step of the call in one workgroup of NW wavefronts.  Lane l of
// wavefront w forms the face left of cell 63 w + l and owns that cell (lane
// 63 owns none), so a cell's right face arrives from the next lane.  A stage then needs one barrier: the owners
// write the next stage's records into the other of two buffers (and the
// ghosts that mirror their cell).  The CFL maximum of a step meets in LDS
// under that barrier; every thread forms dt, by finalize_dt_kernel's rule.
template <int NW, int SPLIT, int HYB, int W>
__global__ __launch_bounds__(NW * 64) void line_steps_kernel(LineStepsArgs s, KGrid g, KPhys ph) {
  constexpr int NC = NW * LW;  // cells at most
  constexpr int P = NC + 8;          // positions k + 3 of the cells k = -3 .. n + 2, faces up to NC
  __shared__ double rec[2][(LNV + 3) * P];
  __shared__ FaceScratch<LNV> scr[NW];
  __shared__ double roe[NW][LNV][64];
  __shared__ double red[NW];
  __shared__ unsigned int redbad[NW];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = g.n[0];
  StepCtl* ctl = s.ctl;
  double time = ctl->t;
  const double te = ctl->t_end;
  unsigned int status = ctl->status, steps = ctl->steps;
  double dt = ctl->dt;
  const int f0 = wave * LW, j = f0 + lane;
  const bool own = lane < LW && j < n;
  unsigned int gh = 0u;  // ghosts that mirror the cell (bit q), with their flips (bit 8 + q)
  if (own && (j < 3 || j >= n - 3)) {
    for (int q = 0; q < 6; ++q) {
      bool flip;
      if (ghost_index(q < 3 ? q - 3 : n + q - 3, n, g.bc_lo[0], g.bc_hi[0], flip) == j)
        gh |= (flip ? 0x101u : 1u) << q;
    }
  }
  double u[LNV], un[LNV];
#pragma unroll
  for (int v = 0; v < LNV; ++v) u[v] = own ? s.U[(long long)v * n + j] : 1.0;
  auto put_records = [&](double* to) {
    if (!own) return;
    LRec<LNV> r;
    make_lrec<LNV>(u, ph, r);
    lane_put<LNV, P>(to + j + 3, r);
    for (unsigned int m = gh; (m & 0x3fu) != 0u; m &= m - 1u) {
      const int q = __builtin_ctz(m);
      LRec<LNV> gr = r;
      if ((gh >> (8 + q)) & 1u) gr.U[1] = -gr.U[1];
      lane_put<LNV, P>(to + (q < 3 ? q : n + q), gr);
    }
  };
  auto fold_cfl = [&]() {  // CFL maximum of u, met in LDS at the next barrier
    double m = 0.0;
    bool bad = false;
    if (own) m = nan_max(m, cfl_speed_u<LNV>(u, ph.gamma, bad));
    const double wm = wave_max(m != m ? __longlong_as_double(0x7ff0000000000000LL) : m);
    const unsigned long long anybad = __ballot(bad);
    if (lane == 0) {
      red[wave] = wm;
      redbad[wave] = anybad != 0ull;
    }
  };
  int cur = 0;
  put_records(rec[0]);
  fold_cfl();
  __syncthreads();
  for (int step = 0; step < s.n_steps; ++step) {
    double smax = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      smax = fmax(smax, red[w]);
      status |= redbad[w];
    }
    dt = s.cfl_dx / smax;
    if (!(time < te) || status != 0u) {
      dt = 0.0;
      break;  // uniform: the clock has stopped
    }
    if (time + dt > te) dt = te - time;
    time = time + dt;
    steps += 1u;
    if (!(dt > 0.0)) break;
#pragma unroll
    for (int v = 0; v < LNV; ++v) un[v] = u[v];
#pragma unroll 1
    for (int st = 0; st < 3; ++st) {
      double ra, rb;
      line_rk(st, ra, rb);
      if (f0 < n) {  // uniform in the wavefront: it owns a cell
        double F60[LNV], dF[LNV], Fr[LNV], dr[LNV];
        const bool m = wave_face<LNV, 0, P, SPLIT, HYB, W>(rec[cur] + f0, 1, j <= n, ph, nullptr, scr[wave], roe[wave], F60, dF);
        const unsigned long long mw = __ballot(m);
#pragma unroll
        for (int v = 0; v < LNV; ++v) {
          Fr[v] = next_lane(F60[v]);
          dr[v] = 0.0;
        }
        if (mw != 0ull) {
#pragma unroll
          for (int v = 0; v < LNV; ++v) dr[v] = next_lane(dF[v]);
        }
        if (own) line_update(u, un, F60, Fr, m, ((mw >> lane) & 2ull) != 0ull, dF, dr, ra, rb, dt, ph);
      }
      cur ^= 1;
      put_records(rec[cur]);
      if (st == 2 && step + 1 < s.n_steps) fold_cfl();
      __syncthreads();
    }
  }
  if (own) {
#pragma unroll
    for (int v = 0; v < LNV; ++v) s.U[(long long)v * n + j] = u[v];
  }
  if (threadIdx.x == 0) {
    ctl->t = time;
    ctl->dt = dt;
    ctl->steps = steps;
    ctl->status = status;
  }
}

// State shared by the launches of one call of the one-launch-per-step form.
// Step i reads the CFL maximum folded into set i mod 3 by the step before and
// the clock i mod 2, folds its own result into set (i + 1) mod 3, writes the
// other clock and clears set (i + 2) mod 3, which the step before read: no
// launch writes what another wavefront of it may still read.
struct LineCtl {
  struct alignas(128) Slot {
    unsigned long long bits;
    unsigned int bad;
  } set[3][CFL_SLOTS];
  struct Clock {
    double t;
    unsigned int steps, status;
  } clk[2];
};

struct LineStepArgs {
  const double* U;  // U^n
  double* out;      // U^(n+1), another array
  LineCtl* lc;
  StepCtl* ctl;     // t_end; dt is recorded
  double cfl_dx, s_floor;
  int i;            // index of the step in the call
  int fold;         // fold the CFL speed of the new state
};

constexpr int LT = 46;       // cells per wavefront: 64 lanes less 9 halo cells a side
constexpr int LHALO = 9;     // 3 stages x 3 cells
constexpr int LP = 72;       // record positions (lane + 3, padded)

// Fold a wavefront's CFL maximum and non-physical flag into its slot.
__device__ __forceinline__ void line_fold(LineCtl::Slot* set, double smax, bool bad) {
  const double m = wave_max(smax != smax ? __longlong_as_double(0x7ff0000000000000LL) : smax);
  const unsigned long long anybad = __ballot(bad);
  const unsigned int wave = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if ((threadIdx.x & 63) == 0) {
    LineCtl::Slot* q = &set[wave % CFL_SLOTS];
    if (m > 0.0) atomicMax(&q->bits, (unsigned long long)__double_as_longlong(m));
    if (anybad) atomicOr(&q->bad, 1u);
  }
}

// LDS of a wavefront's tile.
struct LineShared {
  double rec[(LNV + 3) * LP];
  FaceScratch<LNV> scr;
  double roe[LNV][64];
};

// Index of the cell at line position k of the lane (periodic images wrap,
// positions past the other sides are clamped), and whether it evolves: an
// in-grid cell or a periodic image of one.
__device__ __forceinline__ bool line_cell(const KGrid& g, int k, int& idx) {
  const int n = g.n[0];
  if (g.bc_lo[0] == BC_PERIODIC) {
    idx = k % n;
    if (idx < 0) idx += n;
    return true;
  }
  idx = k < 0 ? 0 : (k >= n ? n - 1 : k);
  return k >= 0 && k < n;
}

// The three stages of one step on the tile of cells x0 .. x0 + LT - 1 (lane l
// holds cell x0 - LHALO + l in u, replaced by its new state).
template <int SPLIT, int HYB, int W>
__device__ __forceinline__ void line_tile(const KGrid& g, const KPhys& ph, int x0, bool cell, double dt,
                                          double (&u)[LNV], LineShared& sh) {
  const int lane = threadIdx.x & 63, n = g.n[0], k = x0 - LHALO + lane;
  const bool per = g.bc_lo[0] == BC_PERIODIC;
  double* rec = sh.rec;
  double un[LNV];
  // ghosts: the lane of the cell they mirror (in the tile wherever the ghost
  // is needed), or the inflow state
  bool flip = false;
  const bool ghost = !cell && k >= -3 && k < n + 3;
  const bool inflow = ghost && k < 0 && g.bc_lo[0] == BC_INFLOW;
  int src = ghost ? ghost_index(k, n, g.bc_lo[0], g.bc_hi[0], flip) - (x0 - LHALO) : 0;
  src = src < 0 ? 0 : (src > 63 ? 63 : src);
  if (inflow) {
    load_inflow<LNV>(g, 0, u);
    flip = false;
  }
#pragma unroll
  for (int v = 0; v < LNV; ++v) un[v] = u[v];
#pragma unroll 1
  for (int st = 0; st < 3; ++st) {
    double ra, rb;
    line_rk(st, ra, rb);
    LRec<LNV> r;
    make_lrec<LNV>(u, ph, r);
    lane_put<LNV, LP>(rec + lane + 3, r);
    wave_lds_fence();
    if (ghost && !inflow) {
      LaneSrc<LNV, LP>{rec + src + 3, 1}.get(0, r);
      if (flip) r.U[1] = -r.U[1];
      lane_put<LNV, LP>(rec + lane + 3, r);
    }
    wave_lds_fence();
    const int lo = 3 * (st + 1), hi = 64 - lo;  // cells updated by this stage
    double F60[LNV], dF[LNV], Fr[LNV], dr[LNV];
    const bool face = lane >= lo && lane <= hi && (per || (k >= 0 && k <= n));
    const bool m = wave_face<LNV, 0, LP, SPLIT, HYB, W>(rec, 1, face, ph, nullptr, sh.scr, sh.roe, F60, dF);
    const unsigned long long mw = __ballot(m);
    const bool mr = ((mw >> lane) & 2ull) != 0ull;
#pragma unroll
    for (int v = 0; v < LNV; ++v) {
      Fr[v] = next_lane(F60[v]);
      dr[v] = 0.0;
    }
    if (mw != 0ull) {
#pragma unroll
      for (int v = 0; v < LNV; ++v) dr[v] = next_lane(dF[v]);
    }
    if (cell && lane >= lo && lane < hi) line_update(u, un, F60, Fr, m, mr, dF, dr, ra, rb, dt, ph);
  }
}

// One step.  Bound: a chain of three stages of ~250 dependent FP64 operations
// each (~750 with WENO faces) on one wavefront per SIMD, plus the launch.
template <int SPLIT, int HYB, int W>
__global__ __launch_bounds__(64) void line_step_kernel(LineStepArgs a, KGrid g, KPhys ph) {
  __shared__ LineShared sh;
  const int lane = threadIdx.x, n = g.n[0];
  const int x0 = blockIdx.x * LT, k = x0 - LHALO + lane;
  int idx;
  const bool cell = line_cell(g, k, idx);
  double u[LNV];
#pragma unroll
  for (int v = 0; v < LNV; ++v) u[v] = a.U[(long long)v * n + idx];
  const bool own = lane >= LHALO && lane < LHALO + LT && k < n;  // cells stored here

  // dt: clock_dt_wave's rule
  LineCtl* lc = a.lc;
  const LineCtl::Slot* in = lc->set[a.i % 3];
  unsigned long long mb = 0ull;
  unsigned int bad_in = 0u;
  if (lane < CFL_SLOTS) {
    mb = in[lane].bits;
    bad_in = in[lane].bad;
  }
  const LineCtl::Clock ck = lc->clk[a.i & 1];
  const double te = a.ctl->t_end;
  double smax = wave_max(__longlong_as_double((long long)mb));  // (no slot holds a NaN)
  if (a.s_floor > smax) smax = a.s_floor;
  const unsigned int status = ck.status | (__ballot(bad_in != 0u) != 0ull ? 1u : 0u);
  double dt = a.cfl_dx / smax;
  const bool stop = !(ck.t < te) || status != 0u;
  if (stop) dt = 0.0;
  else if (ck.t + dt > te) dt = te - ck.t;
  if (blockIdx.x == 0) {
    if (lane < CFL_SLOTS) {
      LineCtl::Slot* clr = &lc->set[(a.i + 2) % 3][lane];
      clr->bits = 0ull;
      clr->bad = 0u;
    }
    if (lane == 0) {
      lc->clk[(a.i + 1) & 1] = LineCtl::Clock{ck.t + dt, ck.steps + (stop ? 0u : 1u), status};
      a.ctl->dt = dt;
    }
  }
  if (!(dt > 0.0)) {  // the clock has stopped: the state passes on unchanged
    if (own) {
#pragma unroll
      for (int v = 0; v < LNV; ++v) a.out[(long long)v * n + k] = u[v];
    }
    return;
  }

  line_tile<SPLIT, HYB, W>(g, ph, x0, cell, dt, u, sh);
  double smx = 0.0;
  bool bad = false;
  if (own) {
#pragma unroll
    for (int v = 0; v < LNV; ++v) a.out[(long long)v * n + k] = u[v];
    if (a.fold) smx = nan_max(smx, cfl_speed_u<LNV>(u, ph.gamma, bad));
  }
  if (a.fold) line_fold(lc->set[(a.i + 1) % 3], smx, bad);
}

// Before the first step: t_end, the clock and empty sets (one wavefront) ...
[[maybe_unused]] static __global__ void line_begin_kernel(LineCtl* lc, StepCtl* ctl, double t_end) {
  const int t = threadIdx.x;
  if (t < CFL_SLOTS) {
    for (int q = 0; q < 3; ++q) {
      lc->set[q][t].bits = 0ull;
      lc->set[q][t].bad = 0u;
    }
  }
  if (t == 0) {
    ctl->t_end = t_end;
    lc->clk[0] = LineCtl::Clock{ctl->t, ctl->steps, ctl->status};
  }
}

// ... then the CFL maximum of U into set 0, and, where the number of steps is
// odd, the copy the first step reads (the last then writes U).
[[maybe_unused]] static __global__ __launch_bounds__(RED_BLOCK) void line_cfl_kernel(
    const double* __restrict__ U, int n, double gamma, LineCtl* lc, double* copy) {
  double smax = 0.0;
  bool bad = false;
  for (int c = blockIdx.x * RED_BLOCK + threadIdx.x; c < n; c += gridDim.x * RED_BLOCK) {
    double u[LNV];
#pragma unroll
    for (int v = 0; v < LNV; ++v) {
      u[v] = U[(long long)v * n + c];
      if (copy != nullptr) copy[(long long)v * n + c] = u[v];
    }
    smax = nan_max(smax, cfl_speed_u<LNV>(u, gamma, bad));
  }
  line_fold(lc->set[0], smax, bad);
}

// After the last of n steps: the clock and status to the control block.
[[maybe_unused]] static __global__ void line_end_kernel(const LineCtl* lc, StepCtl* ctl, int n) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const LineCtl::Clock c = lc->clk[n & 1];
  ctl->t = c.t;
  ctl->steps = c.steps;
  ctl->status = c.status;
}

}  // namespace wl2
