// Batched form: many independent 1D/2D grids advanced by persistent kernels
// walking tables of work items (one table per dimension), so a fixed launch
// shape serves any mix of grid sizes and the per-step launch sequence can be
// captured once in a hipGraph.  A 2D item is a tile of the single-grid tile
// kernel (63 columns x R rows, corrections in place), a 1D item a tile of the
// single-grid line kernel (46 cells, a whole step), with the grid's own dt,
// clock and status, so a run's result is bit-identical to running it alone.
// Bound: the FP64 issue and the chain of a tile, as there; a step is five
// launches (fourteen with a list of flagged cells and a correction kernel per
// stage: 320 us per step for 28 1D and 12 2D runs of 0.65 M cells).
#pragma once
#include "wl2_aux.hpp"
#include "wl2_line.hpp"
#include "wl2_tile.hpp"

namespace wl2 {

// Device-resident descriptor of one admitted grid (one slot).  The arrays are
// element offsets into the pool, which the kernels get as an argument (so
// that they address it as global memory).
struct BGrid {
  KGrid g;
  KPhys ph;
  long long U;   // state U^n, updated in place by the third stage
  long long U1;  // stage buffers
  long long U2;
  double cfl_dx;
  int dim;
};

constexpr int BATCH_MAX_SLOTS = 4096;
constexpr int BATCH_CHUNK = 1024;  // cells per reduction chunk

// Work item: 2D, columns x0 .. x0 + 62 and rows y0 .. of the grid in `slot`;
// 1D, cells x0 .. x0 + 45.
struct BatchItem {
  int slot, x0, y0, pad;
};

// Reduction chunks: chunk c covers cells [first[c], first[c] + count[c]) of
// slot cslot[c].
struct BChunks {
  int n;
  int pad;
  int* cslot;
  long long* first;
  int* count;
};

// Stage STAGE of every 2D run; beside it, in stage 0 the whole step of every
// 1D run (U to U1), in stage 1 its copy back (other items still read U before).
// FAST: every admitted run has the default scheme (LLF splitting, per-field
// switch, Eq.(28)), fixed at compile time; else the build that reads it at run
// time, which spills, serves them all (the same bits; 28 1D and 12 2D runs, us
// per step: all default 165, one 2D run of another scheme 224, all 2D runs 201;
// both codes in one kernel spill as well: 52 us per stage against 48).
template <int R, int STAGE, bool FAST>
__global__ __launch_bounds__((2 * R + 1) * 64, 4) void batch_stage_kernel(
    const BGrid* __restrict__ grids, double* pool, StepCtl* ctls, const BatchItem* __restrict__ items1,
    const BatchItem* __restrict__ items2, const int* __restrict__ n_items) {
  constexpr int NW = 2 * R + 1;
  constexpr size_t BYTES = sizeof(TileShared<R>) > NW * sizeof(LineShared) ? sizeof(TileShared<R>)
                                                                           : NW * sizeof(LineShared);
  __shared__ __attribute__((aligned(16))) char raw[BYTES];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int n1 = STAGE < 2 ? n_items[0] : 0, n1g = (n1 + NW - 1) / NW;  // a 1D item per wavefront
  const int total = n1g + n_items[1];
  for (int q = blockIdx.x; q < total; q += gridDim.x) {
    if (q < n1g) {
      const int i = q * NW + wave;
      if (i < n1) {
        const int slot = items1[i].slot, x0 = items1[i].x0;
        const BGrid& G = grids[slot];
        __builtin_assume(G.g.bc_lo[0] != BC_INFLOW);  // (not admitted)
        const double dt = ctls[slot].dt;
        if (dt > 0.0) {  // else a finished (or not started) run
          const int n = G.g.n[0], k = x0 - LHALO + lane;
          const bool own = lane >= LHALO && lane < LHALO + LT && k < n;
          double* U = pool + G.U;
          double* U1 = pool + G.U1;
          double u[LNV];
          if (STAGE == 0) {
            int idx;
            const bool cell = line_cell(G.g, k, idx);
#pragma unroll
            for (int v = 0; v < LNV; ++v) u[v] = U[(long long)v * n + idx];
            LineShared& sh = reinterpret_cast<LineShared*>(raw)[wave];
            line_tile<FAST ? SPLIT_LLF : -1, FAST ? HYB_PER_FIELD : -1, FAST ? W_L2IS : -1>(G.g, G.ph, x0, cell,
                                                                                          dt, u, sh);
            if (own) {
#pragma unroll
              for (int v = 0; v < LNV; ++v) U1[(long long)v * n + k] = u[v];
            }
          } else if (own) {
#pragma unroll
            for (int v = 0; v < LNV; ++v) U[(long long)v * n + k] = U1[(long long)v * n + k];
          }
        }
      }
    } else {
      const BatchItem it = items2[q - n1g];
      const BGrid& G = grids[it.slot];
      // a finished run that waits to be fetched loads nothing (asked for beside
      // its descriptor: all 40 runs of a mix finished, 73 -> 29 us per step)
      if (ctls[it.slot].dt > 0.0) {
        const KGrid g = G.g;
        const KPhys ph = G.ph;
        __builtin_assume(g.bc_lo[0] != BC_INFLOW);  // (not admitted)
        TileArgs ta{};
        ta.r.Uk = pool + (STAGE == 0 ? G.U : (STAGE == 1 ? G.U1 : G.U2));
        ta.r.out = pool + (STAGE == 0 ? G.U1 : (STAGE == 1 ? G.U2 : G.U));
        ta.r.Un = pool + G.U;
        ta.r.ctl = ctls + it.slot;
        ta.r.rk_a = STAGE == 0 ? 0.0 : (STAGE == 1 ? 0.75 : 1.0 / 3.0);
        ta.r.rk_b = STAGE == 0 ? 1.0 : (STAGE == 1 ? 0.25 : 2.0 / 3.0);
        TileShared<R>& sh = *reinterpret_cast<TileShared<R>*>(raw);
        tile2d_item<R, OUT_RK, FAST ? SPLIT_LLF : -1, FAST ? HYB_PER_FIELD : -1, FAST ? W_L2IS : -1>(
            ta, g, ph, it.x0, it.y0, false, sh);
      }
    }
    __syncthreads();  // the LDS is free for the next item
  }
}

// Per-grid CFL maximum over reduction chunks; one atomic per chunk.  The
// per-cell arithmetic is the same as cfl_reduce_kernel (bit-identical dt).
static __global__ __launch_bounds__(RED_BLOCK) void batch_cfl_kernel(const BGrid* __restrict__ grids,
                                                                     const double* pool, StepCtl* ctl,
                                                                     BChunks ch, const int* nchunks) {
#pragma clang fp contract(off)
  __shared__ double sh[RED_BLOCK / 64];
  const int n = *nchunks;
  for (int c = blockIdx.x; c < n; c += gridDim.x) {
    const BGrid& G = grids[ch.cslot[c]];
    const long long c0 = ch.first[c];
    const int cnt = ch.count[c];
    const long long nc = G.g.ncell;
    const double* U = pool + G.U;
    const double gamma = G.ph.gamma;
    double smax = 0.0;
    bool bad = false;
    for (int q = threadIdx.x; q < cnt; q += RED_BLOCK) {
      const long long cc = c0 + q;
      if (G.dim == 1) {
        const double m[1] = {U[nc + cc]};
        smax = nan_max(smax, cfl_speed<1>(U[cc], m, U[2 * nc + cc], gamma, bad));
      } else {
        const double m[2] = {U[nc + cc], U[2 * nc + cc]};
        smax = nan_max(smax, cfl_speed<2>(U[cc], m, U[3 * nc + cc], gamma, bad));
      }
    }
    const double bm = block_max(smax, sh);
    if (threadIdx.x == 0 && (bm > 0.0 || bm != bm)) cfl_fold(ctl + ch.cslot[c], bm);
    if (bad) atomicOr(&ctl[ch.cslot[c]].status, 1u);
  }
}

// One wavefront per active slot: dt from its maximum, clipped to its own t_end
// (dt = 0 once finished or after a non-physical state).
[[maybe_unused]] static __global__ __launch_bounds__(64) void batch_finalize_kernel(
    const BGrid* __restrict__ grids, StepCtl* ctls, const int* slots, const int* nslots) {
  const int n = *nslots;
  for (int i = blockIdx.x; i < n; i += gridDim.x) {
    StepCtl* ctl = ctls + slots[i];
    double dt = grids[slots[i]].cfl_dx / cfl_take_wave(ctl);
    if (threadIdx.x != 0) continue;
    const double t = ctl->t, te = ctl->t_end;
    if (!(t < te) || ctl->status != 0u || !(dt > 0.0)) {
      dt = 0.0;
    } else {
      if (t + dt > te) dt = te - t;
      ctl->t = t + dt;
      ctl->steps += 1u;
    }
    ctl->dt = dt;
  }
}

// Snapshot of every active slot's clock and status for the host poll.
struct SlotState {
  double t, t_end;
  unsigned int status;
  int slot;
};

[[maybe_unused]] static __global__ void batch_gather_kernel(const StepCtl* ctls, const int* slots,
                                    const int* nslots, SlotState* out) {
  const int n = *nslots;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const StepCtl* ctl = ctls + slots[i];
    out[i].t = ctl->t;
    out[i].t_end = ctl->t_end;
    out[i].status = ctl->status;
    out[i].slot = slots[i];
  }
}

}  // namespace wl2
