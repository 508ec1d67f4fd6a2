// Fused 1D/2D stage kernel (gfx950, FP64): both sweep directions, the flux
// difference of Eq.(19) and the SSP-RK3 stage combination in one pass over
// HBM.
//
// Work item: one wavefront owns RT = 63 consecutive columns of one grid and
// marches along y through a chunk of rows (1D: the single row).  Each lane
// keeps a six-cell window of light records (U, p, c, 1/sqrt(rho)) of its
// column, four in registers and the two oldest in an LDS ring, so the y face
// of every row is formed without another load.  The current row plus a
// three-cell x halo is staged in LDS; lane t computes the x face on the left
// of column t (64 faces for 63 cells) and the right face of a cell arrives
// from the next lane by a lane move, so every face flux is computed
// once and both neighbours use the same bits.  Faces whose detector asks for
// the nonlinear flux are only flagged in the march: their cells go to a
// correction list and a separate kernel adds the WENO-L2IS part (one thread
// per listed cell, so a discontinuity does not serialise the item that holds
// it).  Rows are read with coalesced loads; the next row of the window and of
// the halo is prefetched a row ahead, with the sign flip of mirror ghosts
// applied at use.
#pragma once
#include "wl2_aux.hpp"
#include "wl2_lface.hpp"
#include "wl2_wface.hpp"

namespace wl2 {

constexpr int RW = 64;      // lanes of a work item (one wavefront)
constexpr int RT = RW - 1;  // columns owned by an item: RW x faces
constexpr int RB = RW + 5;  // row buffer: cells x0-3 .. x0+RW+1

struct RowArgs {
  const double* Uk;    // stage input
  double* out;         // RK: U^(k+1); WRITE: dU/dt
  const double* Un;    // RK: U^n (read when rk_a != 0)
  StepCtl* ctl;        // dt and the global LF speeds
  double rk_a, rk_b;   // RK: out = rk_a U^n + rk_b (Uk + dt dU)
  unsigned long long* list;  // cells next to a face that needs the WENO flux
  unsigned int* list_n;      // entries in list
  unsigned int* list_clear;  // if set: the next stage's counter, zeroed by the
                             // correction kernel
  StepCtl* cfl;              // RK: if set, fold the CFL speed of the new state
                             // into cfl->smax / status (next step's dt)
  StepCtl* clock;            // RK stage 1 of a step whose CFL maximum the step
                             // before folded: the stage kernel forms the step's
                             // dt itself (clock_dt_wave, with cfl_dx and the
                             // inflow speed floor s_floor) and its correction
                             // kernel commits the clock (clock_commit); else null
  double cfl_dx, s_floor;
  // LF splitting within a call of several stages: the speeds that the stage
  // before folded (null: ctl->lf_bits holds them), where those of the output are
  // folded (or null), and the set to clear for the next stage.  Against a
  // reduction pass and its finalisation per stage (14.5 + 4.6 us at 1531x1013):
  // 238 -> 212 us per step
  const LfSlot* lf_in;
  LfSlot* lf_out;
  LfSlot* lf_clear;
};

// What a kernel folds from the cells that it finishes: the CFL speed (a.cfl)
// and, in builds that may split globally, the LF speeds (a.lf_out).
template <int NV, bool LF>
struct CellFold {
  double cfl_max = 0.0, mx[LF ? NV - 2 : 1][3] = {};
  bool cfl_bad = false;
  __device__ __forceinline__ void cell(const RowArgs& a, const KPhys& ph, const double (&un)[NV]) {
    if (a.cfl != nullptr) cfl_max = nan_max(cfl_max, cfl_speed_u<NV>(un, ph.gamma, cfl_bad));
    if constexpr (LF) {
      if (a.lf_out != nullptr) lf_fold_cell<NV>(un, ph.gamma, mx);
    }
  }
  __device__ __forceinline__ void commit(const RowArgs& a) {
    if (a.cfl != nullptr) cfl_commit_wave(a.cfl, cfl_max, cfl_bad);
    if constexpr (LF) {
      if (a.lf_out != nullptr) lf_commit_wave<NV - 2>(a.lf_out, mx);
    }
  }
};
template <int NV, int OUT, int SPLIT>
constexpr bool folds_lf() { return NV == 4 && OUT == OUT_RK && (SPLIT < 0 || SPLIT == SPLIT_LF); }

// Entry of the correction list: element offset << 8 | face mask (bit 0 x-, 1
// x+, 2 y-, 3 y+).  A wavefront collects its entries in LDS (buf, n of them)
// and moves them to the list with one atomic when LIST_BUF fills up and at
// the end of its item: an atomic per row, all on one counter, had each
// wavefront on a shock wait for one round trip per row (33 -> 42 us per stage
// at 1024^2).
constexpr int LIST_BUF = 256;

__device__ __forceinline__ void list_flush(const RowArgs& a, unsigned long long* buf, int& n) {
  if (n == 0) return;
  const int lane = threadIdx.x & (RW - 1);
  unsigned int base = 0;
  if (lane == 0) base = atomicAdd(a.list_n, (unsigned int)n);
  base = (unsigned int)__builtin_amdgcn_readfirstlane((int)base);
  wave_lds_fence();
  for (int i = lane; i < n; i += RW) a.list[base + i] = buf[i];
  wave_lds_fence();
  n = 0;
}

__device__ __forceinline__ void list_append(const RowArgs& a, unsigned long long* buf, int& n, long long off,
                                            unsigned cm) {
  const unsigned long long ball = __ballot(cm != 0u);
  if (!ball) return;
  const int lane = threadIdx.x & (RW - 1);
  const int rank = __popcll(ball & ((1ull << lane) - 1ull));
  if (cm) buf[n + rank] = ((unsigned long long)off << 8) | cm;
  n += __popcll(ball);
  if (n > LIST_BUF - RW) list_flush(a, buf, n);
}

template <int NV>
__device__ __forceinline__ void row_put(double (*buf)[RB], int i, const LRec<NV>& r) {
#pragma unroll
  for (int v = 0; v < NV; ++v) buf[v][i] = r.U[v];
  buf[NV][i] = r.p;
  buf[NV + 1][i] = r.c;
  buf[NV + 2][i] = r.iw;
}

template <int NV>
struct RowSrc {  // six cells of the row buffer from `base`
  double (*buf)[RB];
  int base;
  __device__ __forceinline__ void get(int m, LRec<NV>& r) const {
    const int i = base + m;
#pragma unroll
    for (int v = 0; v < NV; ++v) r.U[v] = buf[v][i];
    r.p = buf[NV][i];
    r.c = buf[NV + 1][i];
    r.iw = buf[NV + 2][i];
  }
};

// Per-lane ring of the two oldest cells of the y window: [2][NV+3][RW].
template <int NV>
__device__ __forceinline__ void ring_put(double (*ring)[NV + 3][RW], int slot, int lane,
                                         const LRec<NV>& r) {
#pragma unroll
  for (int v = 0; v < NV; ++v) ring[slot][v][lane] = r.U[v];
  ring[slot][NV][lane] = r.p;
  ring[slot][NV + 1][lane] = r.c;
  ring[slot][NV + 2][lane] = r.iw;
}

template <int NV>
struct RingSrc {  // y stencil: cells j-2, j-1 from the ring, j .. j+3 registers
  double (*ring)[NV + 3][RW];
  int slot0, slot1, lane;
  const LRec<NV>&r0, &r1, &r2, &r3;
  __device__ __forceinline__ void ring_get(int slot, LRec<NV>& r) const {
#pragma unroll
    for (int v = 0; v < NV; ++v) r.U[v] = ring[slot][v][lane];
    r.p = ring[slot][NV][lane];
    r.c = ring[slot][NV + 1][lane];
    r.iw = ring[slot][NV + 2][lane];
  }
  __device__ __forceinline__ void get(int m, LRec<NV>& r) const {
    if (m == 0) ring_get(slot0, r);
    else if (m == 1) ring_get(slot1, r);
    else r = m == 2 ? r0 : m == 3 ? r1 : m == 4 ? r2 : r3;
  }
};

template <int NV>
struct Win6Src {  // six records in registers
  const LRec<NV> (&w)[6];
  __device__ __forceinline__ void get(int m, LRec<NV>& r) const { r = w[m]; }
};

// Row iy (in the grid) of the column at x: the row's address is uniform in the
// wavefront and the column a 32-bit byte offset (nx <= ROW_MAX_NX: wider grids,
// of which those of two and three rows fit the device, take the tile kernel).
template <int NV>
__device__ __forceinline__ void row_load_in(const double* __restrict__ U, const KGrid& g, unsigned x8, int iy,
                                            double (&u)[NV]) {
  const char* p = (const char*)(U + (long long)iy * g.stride[1]);
#pragma unroll
  for (int v = 0; v < NV; ++v) u[v] = *(const double*)(p + v * g.ncell * 8 + x8);
}

// Raw cell (column element offset xy, row y) of a 2D grid, ghost-mapped in
// y; the mirror flip of the y momentum is reported, not applied.
template <int NV>
__device__ __forceinline__ void row_load_raw(const double* __restrict__ U, const KGrid& g,
                                             long long xy, int y, double (&u)[NV]) {
  bool fy = false;
  const int iy = (y >= 0 && y < g.n[1]) ? y : ghost_clamped(y, g.n[1], g.bc_lo[1], g.bc_hi[1], fy);
  const long long off = xy + (long long)iy * g.stride[1];
#pragma unroll
  for (int v = 0; v < NV; ++v) u[v] = U[v * g.ncell + off];
  // state ghosts of a y side (2D grids: xy is the column's x)
  if (NV == 4 && (y < 0 || y >= g.n[1]) && is_yghost(g, y)) load_yghost<NV>(g, xy, y, u);
}

template <int NV>
__device__ __forceinline__ void row_flip(const KGrid& g, bool fx, int y, double (&u)[NV]) {
  bool fy = false;
  if (NV >= 4 && (y < 0 || y >= g.n[1])) (void)ghost_clamped(y, g.n[1], g.bc_lo[1], g.bc_hi[1], fy);
  if (fx) u[1] = -u[1];
  if (NV >= 4 && fy) u[2] = -u[2];
}

// One work item: columns x0 .. x0+RT-1 (clipped to the grid), rows y0 .. y1-1
// (1D: y0 = 0, y1 = 1): the linear-branch fluxes of all its faces, Eq.(19)
// and the stage combination; cells next to a flagged face are listed.
// Called by whole wavefronts; `buf` is the item's LDS row buffer [NV+3][RB],
// `ring` its window ring [2][NV+3][RW] (2D), `lbuf` its list entries.
template <int NV, int OUT, int SPLIT, int HYB>
__device__ __forceinline__ void row_item(const RowArgs& a, const KGrid& g, const KPhys& ph,
                                         double (*buf)[RB], double (*ring)[NV + 3][RW],
                                         unsigned long long* lbuf, int x0, int y0, int y1, double dt) {
  int ln = 0;  // entries in lbuf
  const int lane = threadIdx.x & (RW - 1);
  // global LF speeds, x and y (read only by LF builds)
  unsigned long long lfx[NV], lfy[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    lfx[k] = a.ctl->lf_bits[0][k];
    lfy[k] = a.ctl->lf_bits[1][k];
  }
  constexpr bool LF = folds_lf<NV, OUT, SPLIT>();
  if constexpr (LF) {
    if (a.lf_in != nullptr) {
      lf_take_wave<NV>(a.lf_in, 0, lfx);
      lf_take_wave<NV>(a.lf_in, 1, lfy);
      if (blockIdx.x == 0 && lane < LF_SLOTS) a.lf_clear[lane] = LfSlot{};
      if (blockIdx.x == 0 && lane == 0) {  // for the correction kernels
#pragma unroll
        for (int k = 0; k < NV; ++k) {
          a.ctl->lf_bits[0][k] = lfx[k];
          a.ctl->lf_bits[1][k] = lfy[k];
        }
      }
    }
  }
  // the lane's column (a ghost or the next item's column for lane RT and past
  // the grid edge: those fill the row buffer but own no cell)
  bool fx;
  const int cx = ghost_clamped(x0 + lane, g.n[0], g.bc_lo[0], g.bc_hi[0], fx);
  const bool own = lane < RT && x0 + lane < g.n[0];
  // halo cells: lanes 0-2 fill slots 0-2 (x0-3 .. x0-1), lanes 3-4 slots
  // RW+3, RW+4 (x0+RW, x0+RW+1)
  const bool halo = lane < 5;
  const int hslot = lane < 3 ? lane : RW + lane;
  bool fxh = false;
  const int hx = halo ? ghost_clamped(x0 - 3 + hslot, g.n[0], g.bc_lo[0], g.bc_hi[0], fxh) : 0;
  // halo ghost of an inflow side: its state comes from g.inflow
  const bool hin = halo && x0 - 3 + hslot < 0 && g.bc_lo[0] == BC_INFLOW;
  const long long oxy = cx;  // row 0 element offset of the column (x stride 1)
  const long long hxy = hx;
  const unsigned cx8 = (unsigned)cx * 8u, hx8 = (unsigned)hx * 8u;
  CellFold<NV, LF> fold;  // of the cells written here

  if constexpr (NV == 3) {
    // 1D: one row
    double u[NV];
    row_load_raw<NV>(a.Uk, g, oxy, 0, u);
    row_flip<NV>(g, fx, 0, u);
    LRec<NV> own_rec;
    make_lrec<NV>(u, ph, own_rec);
    row_put<NV>(buf, lane + 3, own_rec);
    if (halo) {
      double hu[NV];
      row_load_raw<NV>(a.Uk, g, hxy, 0, hu);
      row_flip<NV>(g, fxh, 0, hu);
      if (hin) load_inflow<NV>(g, 0, hu);
      LRec<NV> hr;
      make_lrec<NV>(hu, ph, hr);
      row_put<NV>(buf, hslot, hr);
    }
    double unp[NV] = {};
    if (OUT == OUT_RK && a.rk_a != 0.0) {
#pragma unroll
      for (int v = 0; v < NV; ++v) unp[v] = __builtin_nontemporal_load(&a.Un[v * g.ncell + oxy]);
    }
    __syncthreads();
    double Fx[NV];
    const bool mx =
        face_linear_l<NV, 0, SPLIT, HYB>(RowSrc<NV>{buf, lane}, ph, ph.eps_thr[0], lfx, Fx);
    double Fr[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) Fr[v] = next_lane(Fx[v]);
    const int mxr = next_lane_int((int)mx);
    const unsigned cm = own ? ((mx ? 1u : 0u) | (mxr ? 2u : 0u)) : 0u;
    list_append(a, lbuf, ln, oxy, cm);
    if (own) {
      double un[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const double dU = (Fx[v] - Fr[v]) * ph.inv_dx60;
        if (OUT == OUT_RK) {
          double r = a.rk_b * (own_rec.U[v] + dt * dU);
          if (a.rk_a != 0.0) r += a.rk_a * unp[v];
          __builtin_nontemporal_store(r, &a.out[v * g.ncell + oxy]);
          un[v] = r;
        } else {
          __builtin_nontemporal_store(dU, &a.out[v * g.ncell + oxy]);
        }
      }
      // a listed cell is finished (and its CFL speed counted) by the
      // correction kernel
      if (OUT == OUT_RK && cm == 0u) fold.cell(a, ph, un);
    }
    __syncthreads();  // the buffer is reused by the next item
  } else {
    // 2D: column window = cells y-2, y-1 (LDS ring, slot = row & 1) and
    // y .. y+3 (registers r0..r3) at the top of row y
    LRec<NV> r0, r1, r2, r3;
    double Fyp[NV];
    double upre[NV], hpre[NV];
    bool yprev;  // face y - 1/2 needs the nonlinear flux
    {
      LRec<NV> cm3, cm2, cm1;
      double u[NV];
      row_load_raw<NV>(a.Uk, g, oxy, y0 - 3, u);
      row_flip<NV>(g, fx, y0 - 3, u);
      make_lrec<NV>(u, ph, cm3);
      row_load_raw<NV>(a.Uk, g, oxy, y0 - 2, u);
      row_flip<NV>(g, fx, y0 - 2, u);
      make_lrec<NV>(u, ph, cm2);
      row_load_raw<NV>(a.Uk, g, oxy, y0 - 1, u);
      row_flip<NV>(g, fx, y0 - 1, u);
      make_lrec<NV>(u, ph, cm1);
      row_load_raw<NV>(a.Uk, g, oxy, y0, u);
      row_flip<NV>(g, fx, y0, u);
      make_lrec<NV>(u, ph, r0);
      row_load_raw<NV>(a.Uk, g, oxy, y0 + 1, u);
      row_flip<NV>(g, fx, y0 + 1, u);
      make_lrec<NV>(u, ph, r1);
      row_load_raw<NV>(a.Uk, g, oxy, y0 + 2, u);
      row_flip<NV>(g, fx, y0 + 2, u);
      make_lrec<NV>(u, ph, r2);
      row_load_raw<NV>(a.Uk, g, oxy, y0 + 3, u);
      row_flip<NV>(g, fx, y0 + 3, u);
      make_lrec<NV>(u, ph, r3);
      ring_put<NV>(ring, (y0 - 2) & 1, lane, cm2);
      ring_put<NV>(ring, (y0 - 1) & 1, lane, cm1);
      // face y0 - 1/2: cells y0-3 .. y0+2
      const LRec<NV> wp[6] = {cm3, cm2, cm1, r0, r1, r2};
      yprev = face_linear_l<NV, 1, SPLIT, HYB>(Win6Src<NV>{wp}, ph, ph.eps_thr[1], lfy, Fyp);
      if (halo) row_load_in<NV>(a.Uk, g, hx8, y0, hpre);
    }
    bool fyn = false;  // the prefetched cell is a mirror ghost
    auto prefetch = [&](int y) {
      fyn = false;
      if (y < g.n[1]) {
        row_load_in<NV>(a.Uk, g, cx8, y, upre);
      } else {  // past the grid (uniform)
        const int iy = ghost_clamped(y, g.n[1], g.bc_lo[1], g.bc_hi[1], fyn);
        row_load_in<NV>(a.Uk, g, cx8, iy, upre);
        if (NV == 4 && is_yghost(g, y)) load_yghost<NV>(g, oxy, y, upre);
      }
    };
    double res[NV];  // results of row y - 1
    const auto store_res = [&](int y) {
      char* p = (char*)(a.out + (long long)y * g.stride[1]);
#pragma unroll
      for (int v = 0; v < NV; ++v) __builtin_nontemporal_store(res[v], (double*)(p + v * g.ncell * 8 + cx8));
    };
    for (int y = y0; y < y1; ++y) {
      // Records of what the last row loaded, halo and own, then the loads,
      // then the stores of the last row: a wait stands behind branches the
      // compiler cannot count and waits for everything outstanding, so
      // nothing new may be on its way then (1024^2 163 -> 157 us per step,
      // 1531x1013 with global LF 212 -> 200).
      if (halo) {
        if (fxh) hpre[1] = -hpre[1];
        if (hin) load_inflow<NV>(g, y, hpre);
        LRec<NV> hr;
        make_lrec<NV>(hpre, ph, hr);
        row_put<NV>(buf, hslot, hr);
      }
      if (y > y0) {
        // retire cell y-1 into the ring (over cell y-3), shift, make cell y+3
        ring_put<NV>(ring, (y - 1) & 1, lane, r0);
        r0 = r1;
        r1 = r2;
        r2 = r3;
        if (fx) upre[1] = -upre[1];
        if (fyn) upre[2] = -upre[2];
        make_lrec<NV>(upre, ph, r3);
        // The components that no flip rewrites move to registers of the record
        // by an instruction the compiler cannot fold: it would otherwise keep
        // them where they are, load the next cell elsewhere and copy that at
        // the end of the row, waiting for the load.
        asm volatile("v_mov_b64 %0, %1" : "=v"(r3.U[0]) : "v"(upre[0]));
        asm volatile("v_mov_b64 %0, %1" : "=v"(r3.U[NV - 1]) : "v"(upre[NV - 1]));
      }
      row_put<NV>(buf, lane + 3, r0);  // cell (x, y)
      asm volatile("" ::"v"(r3.U[0]), "v"(r3.U[NV - 1]), "v"(r3.p), "v"(r3.c), "v"(r3.iw)
                   : "memory");  // the loads below stay after these uses
      prefetch(y + 4);
      if (halo) row_load_in<NV>(a.Uk, g, hx8, min(y + 1, g.n[1] - 1), hpre);  // (past the chunk: unused)
      const long long row = (long long)y * g.stride[1], off = oxy + row;
      double unp[NV] = {};
      if (OUT == OUT_RK && a.rk_a != 0.0) {
        const char* p = (const char*)(a.Un + row);
#pragma unroll
        for (int v = 0; v < NV; ++v)
          unp[v] = __builtin_nontemporal_load((const double*)(p + v * g.ncell * 8 + cx8));
      }
      if (own && y > y0) store_res(y - 1);
      __syncthreads();
      __builtin_amdgcn_s_setprio(0);
      // x face on the left of column x0+lane (cells x-3 .. x+2 = slots lane .. lane+5)
      double Fx[NV];
      const bool mx =
          face_linear_l<NV, 0, SPLIT, HYB>(RowSrc<NV>{buf, lane}, ph, ph.eps_thr[0], lfx, Fx);
      // y face y + 1/2: cells y-2, y-1 (ring), y .. y+3 (registers)
      double Fy[NV];
      const bool ycur = face_linear_l<NV, 1, SPLIT, HYB>(
                            RingSrc<NV>{ring, (y - 2) & 1, (y - 1) & 1, lane, r0, r1, r2, r3}, ph,
                            ph.eps_thr[1], lfy, Fy);
      double Fr[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) Fr[v] = next_lane(Fx[v]);
      const int mxr = next_lane_int((int)mx);
      const unsigned cm =
          own ? ((mx ? 1u : 0u) | (mxr ? 2u : 0u) | (yprev ? 4u : 0u) | (ycur ? 8u : 0u)) : 0u;
      list_append(a, lbuf, ln, off, cm);
      yprev = ycur;
      // raised wave priority from the end of a row through the next row's
      // loads and records to its barrier, normal for the faces (measured
      // 1.6 % faster on 2D 1024^2; local to this kernel)
      __builtin_amdgcn_s_setprio(2);
      if (own) {
        double un[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const double dU = ((Fx[v] - Fr[v]) + (Fyp[v] - Fy[v])) * ph.inv_dx60;
          if (OUT == OUT_RK) {
            double r = a.rk_b * (r0.U[v] + dt * dU);
            if (a.rk_a != 0.0) r += a.rk_a * unp[v];
            un[v] = r;
            res[v] = r;
          } else {
            res[v] = dU;
          }
        }
        if (OUT == OUT_RK && cm == 0u) fold.cell(a, ph, un);
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) Fyp[v] = Fy[v];
      __syncthreads();  // row buffer free for the next row
    }
    if (own && y1 > y0) store_res(y1 - 1);
  }
  list_flush(a, lbuf, ln);
  if (OUT == OUT_RK) fold.commit(a);
}

// Nonlinear part of the flux of the flagged faces of one listed cell at
// element offset `off` (face order x-, x+, y-, y+, as in the 3D correction
// kernel), added to the output by one lane; `scale` = rk_b dt for a stage, 1
// for dU/dt; the new state in un.  Each face is recomputed from the stage
// input by both of its cells with the same operations, so both get the same
// bits.
template <int NV, int SPLIT, int HYB>
__device__ __forceinline__ void row_fix_cell(const double* Uk, double* out, const StepCtl* ctl,
                                             const KGrid& g, const KPhys& ph, long long off,
                                             unsigned cm, double scale, double (&un)[NV]) {
  const int x = (int)(off % g.n[0]);
  const int y = (int)(off / g.n[0]);
  double acc[NV];
  serial_correction<NV, SPLIT, HYB>(Uk, g, ph, ctl, x, y, 0, cm, acc);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    un[v] = out[v * g.ncell + off] + scale * (acc[v] * ph.inv_dx);
    out[v * g.ncell + off] = un[v];
  }
}

// Listed cells per workgroup round of the field-parallel mode: the two
// wavefronts of a 2D workgroup take the x and the y faces of 8 cells, one
// lane per (side, field) pair (8 of them); in 1D each takes 8 cells' x faces
// (6 lanes each).
template <int NV>
constexpr int fix_fields_cells() { return NV == 4 ? 8 : 16; }

// Field-parallel corrections of a short list (every cell in flight at once):
// each flagged face's change is formed by NV lanes, one per field
// (face_delta_field), a wavefront running one direction only, so a lane's
// work is the linear face and one field's WENO flux where one lane per face
// runs every flagged field and both directions one after the other.  The
// changes meet in LDS and are summed per cell in the fixed order x-, x+, y-,
// y+ as serial_correction sums them: the same bits.
template <int NV, int OUT, int SPLIT, int HYB>
__device__ __forceinline__ void row_fix_fields(const RowArgs& a, const KGrid& g, const KPhys& ph,
                                               unsigned int n, double scale,
                                               CellFold<NV, folds_lf<NV, OUT, SPLIT>()>& fold) {
  constexpr int NF = 2 * (NV - 2);
  constexpr int CPB = fix_fields_cells<NV>();
  __shared__ double sdf[CPB][NF][NV];
  const int lane = threadIdx.x & 63;
  const int dir = NV == 4 ? (int)(threadIdx.x >> 6) : 0;
  const int cslot = NV == 4 ? (lane >> 3) : (int)(threadIdx.x >> 3);
  const int j = lane & 7, side = j / NV, k = j % NV;
  const int f = 2 * dir + side;
  const bool worker = j < 2 * NV;
  for (unsigned int base = blockIdx.x * CPB; base < n; base += gridDim.x * CPB) {
    const unsigned int i = base + cslot;
    unsigned cm = 0;
    long long off = 0;
    if (i < n) {
      const unsigned long long e = a.list[i];
      off = (long long)((e >> 8) & 0xffffffffull);
      cm = (unsigned)(e & 0xffu);
    }
    double dF[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) dF[v] = 0.0;
    if (worker && ((cm >> f) & 1u)) {
      const int x = (int)(off % g.n[0]), y = (int)(off / g.n[0]);
      const int lane0 = (lane & ~7) + side * NV;
      if (dir == 0) {
        face_delta_field<NV, 0, SPLIT, HYB>(a.Uk, g, ph, a.ctl->lf_bits[0], x, y, 0, side, k, lane0, dF);
      } else {
        if constexpr (NV >= 4)
          face_delta_field<NV, 1, SPLIT, HYB>(a.Uk, g, ph, a.ctl->lf_bits[1], x, y, 0, side, k, lane0, dF);
      }
    }
    if (worker && k == 0) {
#pragma unroll
      for (int v = 0; v < NV; ++v) sdf[cslot][f][v] = dF[v];
    }
    __syncthreads();
    if (threadIdx.x < CPB && base + threadIdx.x < n) {
      const unsigned long long e = a.list[base + threadIdx.x];
      const long long c = (long long)((e >> 8) & 0xffffffffull);
      const unsigned m = (unsigned)(e & 0xffu);
      double acc[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) acc[v] = 0.0;
#pragma unroll
      for (int ff = 0; ff < NF; ++ff) {
        if (!((m >> ff) & 1u)) continue;
        const double sg = (ff & 1) ? -1.0 : 1.0;
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v] += sg * sdf[threadIdx.x][ff][v];
      }
      double un[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        un[v] = a.out[v * g.ncell + c] + scale * (acc[v] * ph.inv_dx);
        a.out[v * g.ncell + c] = un[v];
      }
      if (OUT == OUT_RK) fold.cell(a, ph, un);
    }
    __syncthreads();  // sdf is free for the next round
  }
}

// Single grid.  A list short enough for every cell to be in flight at once
// (launched with 2048 workgroups: 16384 cells in 2D, 32768 in 1D) takes the
// field-parallel mode (latency), a longer one a lane per cell (throughput).
// 128 threads per workgroup.  WPE: wavefronts per SIMD that the registers are
// cut to.  Two hold what a lane keeps (188 to 251 VGPRs); three spill 12 to 40
// bytes of it in 1D, and pay where a lane per cell gives more wavefronts than
// two per SIMD hold: every face WENO, us per right-hand side, two / three,
// 100000 cells 38 / 42, 262000 80 / 79, 400000 122 / 119, 1000000 288 / 282.
template <int NV, int OUT, int SPLIT, int HYB, int WPE>
__global__ __launch_bounds__(128, WPE) void row_fix_kernel(RowArgs a, KGrid g, KPhys ph) {
  // the next stage's list starts empty (no kernel of this stage uses it)
  if (a.list_clear != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *a.list_clear = 0u;
  if (a.clock != nullptr && blockIdx.x == 0 && threadIdx.x == 0) clock_commit(a.clock);
  double scale = 1.0;
  if (OUT == OUT_RK) {
    const double dt = a.ctl->dt;
    if (!(dt > 0.0)) return;
    scale = a.rk_b * dt;
  }
  const unsigned int n = *a.list_n;
  const unsigned int threads = gridDim.x * blockDim.x;
  const unsigned int tid = blockIdx.x * blockDim.x + threadIdx.x;
  CellFold<NV, folds_lf<NV, OUT, SPLIT>()> fold;
  if ((unsigned long long)n <= (unsigned long long)gridDim.x * fix_fields_cells<NV>()) {
    row_fix_fields<NV, OUT, SPLIT, HYB>(a, g, ph, n, scale, fold);
  } else {
    for (unsigned int i = tid; i < n; i += threads) {
      const unsigned long long e = a.list[i];
      double un[NV];
      row_fix_cell<NV, SPLIT, HYB>(a.Uk, a.out, a.ctl, g, ph, (long long)((e >> 8) & 0xffffffffull),
                                   (unsigned)(e & 0xffu), scale, un);
      if (OUT == OUT_RK) fold.cell(a, ph, un);
    }
  }
  if (OUT == OUT_RK) fold.commit(a);
}

// Face-once corrections of a long list (single grid).  Every flagged face
// is shared by two listed cells; the per-cell kernel above computes it for
// each of them.  Here phase A computes, per listed cell, the flagged face
// below it in each direction (x-, y-) once, into D[dir][v][entry], and
// records the cell's entry index in map; phase B sums, per listed cell, its
// flagged faces in the order x-, x+, y-, y+, taking a face above the cell
// from the entry of the cell above it (listed, since the face is flagged)
// or, where that cell is a ghost, computing it.  A face's change of flux has
// the same bits whichever cell computes it, and the sum is the per-cell
// kernel's, so the result is bit-identical.  A list short enough for all of
// its faces' fields to be in flight at once takes phase A field-parallel.
template <int NV, int OUT, int SPLIT, int HYB>
__global__ __launch_bounds__(128) void row_face_kernel(RowArgs a, KGrid g, KPhys ph, double* D,
                                                       unsigned int* map, unsigned int cap) {
  // the next stage's list starts empty (no kernel of this stage uses it)
  if (a.list_clear != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *a.list_clear = 0u;
  if (a.clock != nullptr && blockIdx.x == 0 && threadIdx.x == 0) clock_commit(a.clock);
  if (OUT == OUT_RK && !(a.ctl->dt > 0.0)) return;
  constexpr int ND = NV - 2;
  const unsigned int n = *a.list_n;
  const unsigned int threads = gridDim.x * blockDim.x;
  if ((unsigned long long)ND * n * NV <= threads) {
    // a short list: NV lanes per face, one per field (face_delta_field),
    // every face in flight at once; groups of NV consecutive lanes
    // (direction-major, then entry), so a group never straddles wavefronts
    const unsigned int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ND * n * NV) return;
    const unsigned int q = i / NV, kf = i - q * NV;
    const unsigned int dir = q / n, k = q - dir * n;
    const unsigned long long e = a.list[k];
    const long long off = (long long)((e >> 8) & 0xffffffffull);
    const unsigned cm = (unsigned)(e & 0xffu);
    if (dir == 0 && kf == 0) map[off] = k;
    if (!((cm >> (2 * dir)) & 1u)) return;
    const int x = (int)(off % g.n[0]);
    const int y = (int)(off / g.n[0]);
    const int lane0 = (int)(threadIdx.x & 63) - (int)kf;
    double dF[NV];
    if (dir == 0) {
      face_delta_field<NV, 0, SPLIT, HYB>(a.Uk, g, ph, a.ctl->lf_bits[0], x, y, 0, 0, (int)kf, lane0, dF);
    } else {
      if constexpr (NV >= 4)
        face_delta_field<NV, (NV >= 4 ? 1 : 0), SPLIT, HYB>(a.Uk, g, ph, a.ctl->lf_bits[1], x, y, 0, 0,
                                                            (int)kf, lane0, dF);
    }
    double val = dF[0];
#pragma unroll
    for (int v = 1; v < NV; ++v) val = v == (int)kf ? dF[v] : val;
    D[((size_t)dir * NV + kf) * cap + k] = val;  // lane kf writes value kf
    return;
  }
  // lanes ordered direction-major, so a wavefront takes faces of one direction
  for (unsigned int i = blockIdx.x * blockDim.x + threadIdx.x; i < ND * n; i += threads) {
    const unsigned int dir = i / n, k = i - dir * n;
    const unsigned long long e = a.list[k];
    const long long off = (long long)((e >> 8) & 0xffffffffull);
    const unsigned cm = (unsigned)(e & 0xffu);
    if (dir == 0) map[off] = k;
    if (!((cm >> (2 * dir)) & 1u)) continue;
    const int x = (int)(off % g.n[0]);
    const int y = (int)(off / g.n[0]);
    double dF[NV];
    if (dir == 0) {
      face_delta<NV, 0, SPLIT, HYB>(a.Uk, g, ph, a.ctl->lf_bits[0], x, y, 0, 0, dF);
    } else {
      if constexpr (NV >= 4)
        face_delta<NV, (NV >= 4 ? 1 : 0), SPLIT, HYB>(a.Uk, g, ph, a.ctl->lf_bits[1], x, y, 0, 0, dF);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) D[((size_t)dir * NV + v) * cap + k] = dF[v];
  }
}

template <int NV, int OUT, int SPLIT, int HYB>
__global__ __launch_bounds__(128) void row_sum_kernel(RowArgs a, KGrid g, KPhys ph,
                                                      const double* __restrict__ D,
                                                      const unsigned int* __restrict__ map,
                                                      unsigned int cap) {
  double scale = 1.0;
  if (OUT == OUT_RK) {
    const double dt = a.ctl->dt;
    if (!(dt > 0.0)) return;
    scale = a.rk_b * dt;
  }
  constexpr int ND = NV - 2;
  const unsigned int n = *a.list_n;
  const unsigned int threads = gridDim.x * blockDim.x;
  CellFold<NV, folds_lf<NV, OUT, SPLIT>()> fold;
  for (unsigned int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += threads) {
    const unsigned long long e = a.list[k];
    const long long off = (long long)((e >> 8) & 0xffffffffull);
    const unsigned cm = (unsigned)(e & 0xffu);
    const int x = (int)(off % g.n[0]);
    const int y = (int)(off / g.n[0]);
    double acc[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = 0.0;
#pragma unroll
    for (int f = 0; f < 2 * ND; ++f) {
      if (!((cm >> f) & 1u)) continue;
      const int dir = f >> 1, side = f & 1;
      double d[NV];
      if (side == 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) d[v] = D[((size_t)dir * NV + v) * cap + k];
      } else {
        const int pos = dir == 0 ? x : y;
        if (pos + 1 < g.n[dir]) {
          // the cell above is listed in this stage (its face below is the
          // flagged face); min() only keeps a broken list inside D
          const unsigned int kk = min(map[off + (dir == 0 ? 1ll : g.stride[1])], cap - 1u);
#pragma unroll
          for (int v = 0; v < NV; ++v) d[v] = D[((size_t)dir * NV + v) * cap + kk];
        } else if (dir == 0) {
          face_delta<NV, 0, SPLIT, HYB>(a.Uk, g, ph, a.ctl->lf_bits[0], x, y, 0, 1, d);
        } else {
          if constexpr (NV >= 4)
            face_delta<NV, (NV >= 4 ? 1 : 0), SPLIT, HYB>(a.Uk, g, ph, a.ctl->lf_bits[1], x, y, 0, 1, d);
        }
      }
      const double sg = side ? -1.0 : 1.0;
#pragma unroll
      for (int v = 0; v < NV; ++v) acc[v] += sg * d[v];
    }
    double un[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      un[v] = a.out[v * g.ncell + off] + scale * (acc[v] * ph.inv_dx);
      a.out[v * g.ncell + off] = un[v];
    }
    if (OUT == OUT_RK) fold.cell(a, ph, un);
  }
  if (OUT == OUT_RK) fold.commit(a);
}

[[maybe_unused]] static __global__ void row_list_reset_kernel(unsigned int* n) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *n = 0u;
}

// Single grid: item = (x tile, chunk of `ych` rows), one wavefront each.
template <int NV, int OUT, int SPLIT, int HYB>
__global__ __launch_bounds__(RW, 2) void row_kernel(RowArgs a, KGrid g, KPhys ph, int ych,
                                                    int tiles_x) {
  __shared__ double buf[NV + 3][RB];
  __shared__ double ring[2][NV + 3][RW];
  __shared__ unsigned long long lbuf[LIST_BUF];
  double dt = 0.0;
  if (OUT == OUT_RK) {
    dt = a.clock != nullptr
             ? clock_dt_wave(a.clock, a.cfl_dx, a.s_floor, blockIdx.x == 0 && threadIdx.x == 0)
             : a.ctl->dt;
    if (!(dt > 0.0)) return;  // finished run: leave the state untouched
  }
  const int item = blockIdx.x;
  const int tx = item % tiles_x, ty = item / tiles_x;
  const int y0 = ty * ych;
  const int y1 = min(y0 + ych, g.n[1]);
  row_item<NV, OUT, SPLIT, HYB>(a, g, ph, buf, ring, lbuf, tx * RT, y0, y1, dt);
}

}  // namespace wl2
