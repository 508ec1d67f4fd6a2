// 3D stage with every face WENO: one kernel per direction.
//
// Each face is computed once, its linear flux (times 60) and the change that
// the WENO flux makes to it, and its two cells' differences of both are taken
// where it is computed; the running sums of the directions (five values each)
// pass from kernel to kernel through `part`, and the z kernel finishes the
// cell.  The sums have the order of the stage kernel and its correction kernels
// (x, y, z for the fluxes; x-, x+, y-, y+, z-, z+ for the changes), so the
// results carry their bits.
//
// Bound by FP64 issue (1640 operations per face).  Against a linear stage
// kernel, three kernels that wrote every face's change and one that summed six
// of them per cell, the linear fluxes are formed once instead of twice, 0.66 of
// the 1.98 KB of traffic per cell is gone and the rest is hidden behind the
// arithmetic; along y and z a lane keeps its column's stencil in registers, so
// a face costs one cell's load and record instead of six.  Measured, us per
// stage, before -> now: 160^3 1180 -> 810, 32^3 100 -> 34, 64^3 160 -> 94, 256^3
// 4940 -> 3440 (the weights of Eq.(14)-(15) 6080 -> 3530); splittings other
// than LLF, whose faces were computed for both of their cells, 96^3 489 -> 210.
// The three kernels issue VALU instructions in 91 to 94 % of their cycles, at
// 1.84 to 1.89 GHz; 32 to 36 TFLOP/s at 256^3.
#pragma once
#include "wl2_fused_launch.hpp"
#include "wl2_lface.hpp"

namespace wl2 {

struct Weno3dArgs {
  const double* Uk;
  double* out;
  const double* Un;
  StepCtl* ctl;
  double rk_a, rk_b;
  unsigned int* list_clear;  // the next stage's list counter, zeroed here
  StepCtl* cfl;              // RK: if set, fold the CFL speed of the new state
  double* part;              // [10][cells]: flux differences, then changes
};

constexpr int WX_FACES = 63;  // faces of a wavefront along x whose cell it finishes

// x: the faces of all rows in one index space (nx + 1 per row), 63 per
// wavefront and one more, which the next wavefront computes again; a lane's
// cell lies above its face, the flux on the cell's other side is the next
// lane's.
template <int OUT, int SPLIT, int W>
__global__ __launch_bounds__(64, 2) void weno3d_x_kernel(Weno3dArgs a, KGrid g, KPhys ph) {
  constexpr int NV = 5;
  if (OUT == OUT_RK && !(a.ctl->dt > 0.0)) return;
  const int lane = threadIdx.x;
  const long long rows = (long long)g.n[1] * g.n[2];
  const unsigned nx = (unsigned)g.n[0], ex = nx + 1u;
  const long long i0 = (long long)blockIdx.x * WX_FACES;
  const long long row0 = i0 / ex;  // (uniform)
  const unsigned t = (unsigned)(i0 - row0 * ex) + (unsigned)lane;
  unsigned q = t / ex;
  const int x = (int)(t - q * ex);
  const bool in = row0 + q < rows;
  if (!in) q = (unsigned)(rows - 1 - row0);  // past the last row: any valid row
  // the wavefront's first row by a uniform address, the rest a 32-bit offset
  const char* U = (const char*)(a.Uk + row0 * nx);
  double u[6][NV];
  bool flip[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    const int ix = ghost_clamped(x - 3 + m, g.n[0], g.bc_lo[0], g.bc_hi[0], flip[m]);
    const unsigned o = (q * nx + (unsigned)ix) * 8u;
#pragma unroll
    for (int v = 0; v < NV; ++v) u[m][v] = *(const double*)(U + v * g.ncell * 8 + o);
  }
  LRec<NV> w[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    if (flip[m]) u[m][1] = -u[m][1];
    make_lrec<NV>(u[m], ph, w[m]);
  }
  const WinSrc<NV> src{w[0], w[1], w[2], w[3], w[4], w[5]};
  double F[NV], dF[NV];
  FaceState<NV> st;
  const unsigned mask = face_linear_st<NV, 0, SPLIT, HYB_WENO_ONLY, false>(src, ph, ph.eps_thr[0],
                                                                               a.ctl->lf_bits[0], F, st);
  lean_correction<NV, 0, W>(src, mask, st, F, ph, dF);
  const bool own = lane < WX_FACES && in && x < g.n[0];
  char* p = (char*)(a.part + row0 * nx);
  const unsigned o = (q * nx + (unsigned)x) * 8u;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const double s = F[v] - next_lane(F[v]);
    double acc = 0.0;
    acc += dF[v];
    acc -= next_lane(dF[v]);
    if (own) {
      *(double*)(p + v * g.ncell * 8 + o) = s;
      *(double*)(p + (NV + v) * g.ncell * 8 + o) = acc;
    }
  }
}

// y and z: a lane marches along its column through the cells [k0, k1) of its
// chunk, the six cells of the current face in registers.
template <int OUT, int DIR, int SPLIT, int W>
__global__ __launch_bounds__(64, 2) void weno3d_march_kernel(Weno3dArgs a, KGrid g, KPhys ph,
                                                                         int len, unsigned groups) {
  constexpr int NV = 5;
  __shared__ double prev[2 * NV][64];  // the face below the cell: its flux and change
  if (DIR == 2 && a.list_clear != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *a.list_clear = 0u;
  double dt = 0.0, scale = 1.0;
  if (OUT == OUT_RK) {
    dt = a.ctl->dt;
    if (!(dt > 0.0)) return;
    scale = a.rk_b * dt;
  }
  const long long plane = g.stride[2];
  const long long cols = DIR == 1 ? (long long)g.n[0] * g.n[2] : plane;
  const unsigned chunk = blockIdx.x / groups;
  const long long col = (long long)(blockIdx.x - chunk * groups) * 64 + threadIdx.x;
  const bool own = col < cols;
  const long long c = own ? col : cols - 1;
  const long long coff = DIR == 1 ? c / g.n[0] * plane + c % g.n[0] : c;
  const long long st = DIR == 1 ? g.stride[1] : plane;
  const int n = g.n[DIR];
  const int k0 = (int)chunk * len, k1 = min(k0 + len, n);
  const auto load = [&](int k, double (&u)[NV], bool& flip) {
    const double* p = a.Uk + ghost_clamped(k, n, g.bc_lo[DIR], g.bc_hi[DIR], flip) * st;
#pragma unroll
    for (int v = 0; v < NV; ++v) u[v] = p[v * g.ncell + coff];
  };
  LRec<NV> w[6];
  {
    double u[6][NV];
    bool flip[6];
#pragma unroll
    for (int m = 0; m < 6; ++m) load(k0 - 3 + m, u[m], flip[m]);
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      if (flip[m]) u[m][1 + DIR] = -u[m][1 + DIR];
      make_lrec<NV>(u[m], ph, w[m]);
    }
  }
  // what the cell's end and the next face need is asked for before the last
  // field: its latency passes there, and the registers are free until then
  double nxt[NV], S[NV], A[NV];
  bool fn;
  double cfl_max = 0.0;
  bool cfl_bad = false;
  for (int f = k0; f <= k1; ++f) {
    const WinSrc<NV> src{w[0], w[1], w[2], w[3], w[4], w[5]};
    double F[NV], dF[NV];
    FaceState<NV> fs;
    const unsigned mask = face_linear_st<NV, DIR, SPLIT, HYB_WENO_ONLY, false>(
        src, ph, ph.eps_thr[DIR], a.ctl->lf_bits[DIR], F, fs);
    const long long off = coff + max(f - 1, 0) * st;  // (the first face's is not used)
    double* const part = a.part + off;
    lean_correction<NV, DIR, W>(src, mask, fs, F, ph, dF, [&]() {
      __builtin_amdgcn_sched_barrier(0);
      load(f + 3, nxt, fn);
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        S[v] = part[v * g.ncell];
        A[v] = part[(NV + v) * g.ncell];
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    if (f > k0 && own) {
      double un[NV] = {};
      if (DIR == 2 && OUT == OUT_RK && a.rk_a != 0.0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) un[v] = a.Un[v * g.ncell + off];
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const double s = S[v] + (prev[v][threadIdx.x] - F[v]);
        double acc = A[v];
        acc += prev[NV + v][threadIdx.x];
        acc -= dF[v];
        if (DIR == 1) {
          part[v * g.ncell] = s;
          part[(NV + v) * g.ncell] = acc;
        } else {
          const double dU = s * ph.inv_dx60;
          double r = dU;
          if (OUT == OUT_RK) {
            r = a.rk_b * (w[2].U[v] + dt * dU);
            if (a.rk_a != 0.0) r += a.rk_a * un[v];
          }
          un[v] = r + scale * (acc * ph.inv_dx);
          __builtin_nontemporal_store(un[v], &a.out[v * g.ncell + off]);
        }
      }
      if (DIR == 2 && OUT == OUT_RK && a.cfl != nullptr)
        cfl_max = nan_max(cfl_max, cfl_speed_u<NV>(un, ph.gamma, cfl_bad));
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      prev[v][threadIdx.x] = F[v];
      prev[NV + v][threadIdx.x] = dF[v];
    }
#pragma unroll
    for (int m = 0; m < 5; ++m) w[m] = w[m + 1];
    if (fn) nxt[1 + DIR] = -nxt[1 + DIR];
    make_lrec<NV>(nxt, ph, w[5]);
  }
  if (DIR == 2 && OUT == OUT_RK && a.cfl != nullptr) cfl_commit_wave(a.cfl, cfl_max, cfl_bad);
}

}  // namespace wl2
