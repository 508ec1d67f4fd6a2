// Faces of one wavefront with their corrections in place (gfx950, FP64): the
// linear flux of one face per lane, then the WENO fluxes of the flagged faces
// spread over the wavefront's lanes.  A lane per face would form every field
// that some lane flags, one after the other (and with the few faces a shock
// crosses, on a few lanes); here the (flagged field, face) pairs are numbered
// through and lane i takes the pairs i, i + 64, ..., so up to 64 pairs cost
// one field's WENO flux (spreading them over all wavefronts of a workgroup took
// two more barriers and spilled: 10 to 20 % slower).  Operation for operation the arithmetic of
// face_delta: the same bits.
#pragma once
#include "wl2_lface.hpp"

namespace wl2 {

// Orders the LDS accesses of one wavefront (its lanes exchange values): the
// LDS unit takes them in issue order, the compiler must not reorder them.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Six records in LDS, the first at q, `stride` positions apart; VP: doubles
// between two values of a record.
template <int NV, int VP>
struct LaneSrc {
  const double* q;
  int stride;
  __device__ __forceinline__ void get(int m, LRec<NV>& r) const {
    const double* s = q + m * stride;
#pragma unroll
    for (int v = 0; v < NV; ++v) r.U[v] = s[v * VP];
    r.p = s[NV * VP];
    r.c = s[(NV + 1) * VP];
    r.iw = s[(NV + 2) * VP];
  }
};

template <int NV, int VP>
__device__ __forceinline__ void lane_put(double* q, const LRec<NV>& r) {
#pragma unroll
  for (int v = 0; v < NV; ++v) q[v * VP] = r.U[v];
  q[NV * VP] = r.p;
  q[(NV + 1) * VP] = r.c;
  q[(NV + 2) * VP] = r.iw;
}

// What a lane needs to form one field of another lane's face, and the list of
// (field << 6 | lane) pairs; the Roe state's u, 1/c and 1/rho go to NV rows of
// 64 doubles that the caller names (the rows it keeps the fluxes in
// afterwards), the rest of that state is formed from them again.
template <int NV>
struct FaceScratch {
  double a[3][64];    // splitting speeds of u - c, u, u + c
  double dv[NV][64];  // then the field's WENO flux
  unsigned char pair[NV * 64];
};

// What a flagged face keeps in registers while its fields are formed.
struct FaceKeep {
  double H, c;
};

// Linear flux (times 60) of the lane's face (its first stencil cell at
// rec + lane), and the mask of the fields that need the WENO flux (returned; 0
// for lanes that pass active = false).  Flagged faces leave what face_pair
// needs in the scratch, and the fluxes of their other fields in the place
// where face_pair leaves the WENO fluxes.  total: the wavefront's pairs.
// Called by whole wavefronts.
template <int NV, int DIR, int VP, int SPLIT, int HYB>
__device__ __forceinline__ unsigned face_begin(const double* rec, int stride, bool active, const KPhys& ph,
                                               const unsigned long long* lfb, FaceScratch<NV>& sc,
                                               double (*roe)[64], double (&F60)[NV], FaceKeep& kp,
                                               int& total) {
  constexpr int DIM = NV - 2;
  const int lane = threadIdx.x & 63;
  FaceState<NV> st;
  unsigned mask = face_linear_st<NV, DIR, SPLIT, HYB, false>(LaneSrc<NV, VP>{rec + lane, stride}, ph,
                                                             ph.eps_thr[DIR], lfb, F60, st);
  if (!active) mask = 0u;
  total = 0;
  if (__ballot(mask != 0u) == 0ull) return 0u;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const unsigned long long b = __ballot((mask >> k) & 1u);
    if ((mask >> k) & 1u)
      sc.pair[total + __popcll(b & ((1ull << lane) - 1ull))] = (unsigned char)(k << 6 | lane);
    total += __popcll(b);
  }
  if (mask) {
#pragma unroll
    for (int d = 0; d < DIM; ++d) roe[d][lane] = st.s.u[d];
    roe[DIM][lane] = st.s.ic;
    roe[DIM + 1][lane] = st.s.irho;
    sc.a[0][lane] = st.a[0];
    sc.a[1][lane] = st.a[1];
    sc.a[2][lane] = st.a[NV - 1];
    double LF[NV];
    project<NV, DIR>(st.s, st.Fc6, LF);
#pragma unroll
    for (int k = 0; k < NV; ++k) sc.dv[k][lane] = ((mask >> k) & 1u) ? st.dv[k] : LF[k] + st.a[k] * st.dv[k];
    kp.H = st.s.H;
    kp.c = st.s.c;
  }
  return mask;
}

// One pair e of the wavefront whose faces start at rec: that field's WENO flux
// takes the place of dv in the scratch.
template <int NV, int DIR, int VP, int W>
__device__ __forceinline__ void face_pair(int e, const double* rec, int stride, const KPhys& ph,
                                          FaceScratch<NV>& sc, const double (*roe)[64]) {
  constexpr int DIM = NV - 2;
  const int fl = e & 63, k = e >> 6;
  Roe<NV> s;
  double q = 0.0;  // as in roe_light
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    s.u[d] = roe[d][fl];
    q += s.u[d] * s.u[d];
  }
  s.q = 0.5 * q;
  s.ic = roe[DIM][fl];
  s.irho = roe[DIM + 1][fl];
  s.b1 = ph.gm1 * s.ic * s.ic;
  s.b2 = s.b1 * s.q;
  double r[NV];
  left_row_rt<NV, DIR>(s, k, r);
  const double al = sc.a[k == 0 ? 0 : (k == NV - 1 ? 2 : 1)][fl];
  sc.dv[k][fl] = lean_field_row<NV, DIR, W, -1>(LaneSrc<NV, VP>{rec + fl, stride}, r, s, al, sc.dv[k][fl], ph);
}

// The correction of the lane's flagged face from its fields' fluxes.
template <int NV, int DIR>
__device__ __forceinline__ void face_finish(const FaceKeep& kp, const double (&F60)[NV],
                                            const FaceScratch<NV>& sc, const double (*roe)[64],
                                            double (&dF)[NV]) {
  constexpr int DIM = NV - 2;
  const int lane = threadIdx.x & 63;
  Roe<NV> s;
  double q = 0.0;  // as in roe_light
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    s.u[d] = roe[d][lane];
    q += s.u[d] * s.u[d];
  }
  s.q = 0.5 * q;
  s.H = kp.H;
  s.c = kp.c;
  double f[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) f[k] = sc.dv[k][lane];
  back_project<NV, DIR>(s, f, dF);
#pragma unroll
  for (int v = 0; v < NV; ++v) dF[v] -= F60[v] * (1.0 / 60.0);
}

// All three for one wavefront by itself: dF is the correction of a flagged
// face (returned), else 0.
template <int NV, int DIR, int VP, int SPLIT, int HYB, int W>
__device__ __forceinline__ bool wave_face(const double* rec, int stride, bool active, const KPhys& ph,
                                          const unsigned long long* lfb, FaceScratch<NV>& sc,
                                          double (*roe)[64], double (&F60)[NV], double (&dF)[NV]) {
  FaceKeep kp{};
  int total;
  const unsigned mask = face_begin<NV, DIR, VP, SPLIT, HYB>(rec, stride, active, ph, lfb, sc, roe, F60, kp, total);
#pragma unroll
  for (int v = 0; v < NV; ++v) dF[v] = 0.0;
  if (total == 0) return false;
  wave_lds_fence();
  for (int i = threadIdx.x & 63; i < total; i += 64) face_pair<NV, DIR, VP, W>(sc.pair[i], rec, stride, ph, sc, roe);
  wave_lds_fence();
  if (mask) face_finish<NV, DIR>(kp, F60, sc, roe, dF);
  wave_lds_fence();  // the scratch is free for the wavefront's next faces
  return mask != 0u;
}

}  // namespace wl2
