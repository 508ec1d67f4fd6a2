// Face fluxes from "light" cell records (U, p, c, 1/sqrt(rho)): the linear
// branch of one face, its nonlinear (WENO-L2IS) correction, and the helpers
// they share.  Used by the fused 3D stage kernel and the 1D/2D row kernels;
// stencil cells come through small accessor objects (`src.get(m, rec)`), so
// the same arithmetic serves registers, LDS and global memory.
#pragma once
#include "wl2_device.hpp"

namespace wl2 {

// 1/x and 1/sqrt(x) from the hardware seeds, refined by one third-order step
// (the seed error e is cubed: a seed good to 2^-23 gives 2^-67, below the
// rounding of the last operation; the result is within an ulp or two, not
// correctly rounded).  One operation (rcp) and two (rsqrt) fewer than two
// Newton steps, and a shorter chain.
__device__ __forceinline__ double fast_rcp(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);  // r (1 + e + e^2)
}

__device__ __forceinline__ double fast_rsqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);  // y (1 + e/2 + 3 e^2/8)
}

template <int NV>
struct LRec {
  double U[NV];
  double p, c, iw;  // pressure, sound speed, 1/sqrt(rho)
};

template <int NV>
__device__ __forceinline__ void make_lrec(const double (&u)[NV], const KPhys& ph, LRec<NV>& r) {
  constexpr int DIM = NV - 2;
  const double iw = fast_rsqrt(u[0]);
  // 1/rho corrected to within rounding: at a high Mach number p is a small
  // difference of E and the kinetic energy, and magnifies its error
  const double i2 = iw * iw;
  const double ir = fma(i2, fma(-u[0], i2, 1.0), i2);
  double m2 = 0.0;
#pragma unroll
  for (int k = 0; k < DIM; ++k) m2 += u[1 + k] * u[1 + k];
  const double p = ph.gm1 * (u[NV - 1] - 0.5 * ir * m2);
  const double c2 = ph.gamma * p * ir;
  r.c = c2 * fast_rsqrt(c2);
  r.p = p;
  r.iw = iw;
#pragma unroll
  for (int v = 0; v < NV; ++v) r.U[v] = u[v];
}

// Flux along DIR and normal velocity from a light record.
template <int NV, int DIR>
__device__ __forceinline__ void lflux(const LRec<NV>& r, double (&F)[NV], double& un) {
  constexpr int DIM = NV - 2;
  un = r.U[1 + DIR] * (r.iw * r.iw);
  F[0] = r.U[1 + DIR];
#pragma unroll
  for (int k = 0; k < DIM; ++k) F[1 + k] = un * r.U[1 + k] + (k == DIR ? r.p : 0.0);
  F[NV - 1] = (r.U[NV - 1] + r.p) * un;
}

// Roe average of the two cells at the face; EpL, EpR = E + p of each.  With
// w = sqrt(rho) = 1/iw: 1/(wL + wR) = iwL iwR / (iwL + iwR).
template <int NV, int DIR>
__device__ __forceinline__ void roe_light(const LRec<NV>& L, const LRec<NV>& R, double EpL, double EpR,
                                          const KPhys& ph, Roe<NV>& s) {
  constexpr int DIM = NV - 2;
  s.irho = L.iw * R.iw;
  const double is = s.irho * fast_rcp(L.iw + R.iw);
  const double wl = L.iw * is, wr = R.iw * is;
  double q = 0.0;
#pragma unroll
  for (int k = 0; k < DIM; ++k) {
    s.u[k] = L.U[1 + k] * wl + R.U[1 + k] * wr;
    q += s.u[k] * s.u[k];
  }
  s.q = 0.5 * q;
  s.H = EpL * wl + EpR * wr;
  const double c2 = ph.gm1 * (s.H - s.q);
  s.ic = fast_rsqrt(c2);
  s.c = c2 * s.ic;
  s.b1 = ph.gm1 * s.ic * s.ic;
  s.b2 = s.b1 * s.q;
}

// Intermediate quantities of a linear face that its nonlinear correction
// reuses: the Roe state, the splitting speeds, dv = L dU5 / 60 and Fc6.
template <int NV>
struct FaceState {
  Roe<NV> s;
  double a[NV], dv[NV], Fc6[NV];
};

// The sums over the six stencil cells of a face: dU5 (Eq.(31), times 60), the
// six-point central flux times 60 and the maxima of |u_n - c|, |u_n|,
// |u_n + c|.  A flux is u_n times a conserved value (plus p): the stencil
// weight multiplies u_n once and each flux component is one FMA per cell
// (11 operations per face fewer in 3D than forming every cell's flux and
// weighting it).
template <int NV, int DIR>
struct FaceSums {
  static constexpr int DIM = NV - 2;
  double dU[NV], F[NV], ps, am, a0, ap;

  // Cells a (below the face) and b (above it, mirror position), the weights
  // WF of the flux and WU of U_a - U_b; first: the pair the sums start from.
  template <bool FIRST>
  __device__ __forceinline__ void add(const LRec<NV>& a, const LRec<NV>& b, double WF, double WU,
                                      double& Ea, double& Eb) {
    const double ua = a.U[1 + DIR] * (a.iw * a.iw), ub = b.U[1 + DIR] * (b.iw * b.iw);
    const double m_am = fmax(fabs(ua - a.c), fabs(ub - b.c)), m_a0 = fmax(fabs(ua), fabs(ub)),
                 m_ap = fmax(fabs(ua + a.c), fabs(ub + b.c));
    Ea = a.U[NV - 1] + a.p;
    Eb = b.U[NV - 1] + b.p;
    if (FIRST) {
      am = m_am;
      a0 = m_a0;
      ap = m_ap;
#pragma unroll
      for (int i = 0; i < NV; ++i) dU[i] = a.U[i] - b.U[i];
      F[0] = a.U[1 + DIR] + b.U[1 + DIR];
      ps = a.p + b.p;
#pragma unroll
      for (int k = 0; k < DIM; ++k) F[1 + k] = ua * a.U[1 + k] + ub * b.U[1 + k];
      F[NV - 1] = ua * Ea + ub * Eb;
    } else {
      am = fmax(am, m_am);
      a0 = fmax(a0, m_a0);
      ap = fmax(ap, m_ap);
#pragma unroll
      for (int i = 0; i < NV; ++i) dU[i] += WU * (a.U[i] - b.U[i]);
      F[0] += WF * (a.U[1 + DIR] + b.U[1 + DIR]);
      ps += WF * (a.p + b.p);
      const double wa = WF * ua, wb = WF * ub;
#pragma unroll
      for (int k = 0; k < DIM; ++k) {
        F[1 + k] += wa * a.U[1 + k];
        F[1 + k] += wb * b.U[1 + k];
      }
      F[NV - 1] += wa * Ea;
      F[NV - 1] += wb * Eb;
    }
  }
};

// Linear-branch flux of one face from six light records, with its state for
// a correction, times 60 (the flux difference takes the 1/60 with 1/dx:
// KPhys::inv_dx60).  Cells are requested in the pairs (0,5), (1,4), (2,3) so
// only two are live at a time.  ANY: returns whether the detector of some
// field asks for the nonlinear flux (the largest |dv| decides: the square of
// a product is monotonic in it, so for finite values this agrees with the mask
// bit for bit; a face with a NaN among them has a NaN flux, listed or not);
// else the mask of those fields.
// The dissipation R (alpha dv): the entropy and shear fields share one
// splitting speed a0 and sum_s R^s L^s = 1, so it is a0 dU5 plus the two
// acoustic fields' (alpha - a0) dv (15 operations in place of 25).
template <int NV, int DIR, int SPLIT, int HYB, bool ANY, class Src>
__device__ __forceinline__ unsigned face_linear_st(const Src& src, const KPhys& ph, double eps_thr,
                                                   const unsigned long long* lfb, double (&F60)[NV],
                                                   FaceState<NV>& st) {
  constexpr int DIM = NV - 2;
  const int split = SPLIT >= 0 ? SPLIT : ph.split;
  const int hybrid = HYB >= 0 ? HYB : ph.hybrid;
  FaceSums<NV, DIR> f;
  double Ea, Eb;
  {
    LRec<NV> c0, c5;
    src.get(0, c0);
    src.get(5, c5);
    f.template add<true>(c0, c5, 1.0, 1.0, Ea, Eb);
  }
  {
    LRec<NV> c1, c4;
    src.get(1, c1);
    src.get(4, c4);
    f.template add<false>(c1, c4, -8.0, -5.0, Ea, Eb);
  }
  LRec<NV> c2, c3;
  src.get(2, c2);
  src.get(3, c3);
  f.template add<false>(c2, c3, 37.0, 10.0, Ea, Eb);
  f.F[1 + DIR] += f.ps;
  Roe<NV> s;
  roe_light<NV, DIR>(c2, c3, Ea, Eb, ph, s);
  double am = f.am, a0 = f.a0, ap = f.ap;
  if (split == SPLIT_ROE) {
    am = fabs(s.u[DIR] - s.c);
    a0 = fabs(s.u[DIR]);
    ap = fabs(s.u[DIR] + s.c);
  } else if (split != SPLIT_LLF) {
    am = __longlong_as_double((long long)lfb[0]);
    a0 = __longlong_as_double((long long)lfb[1]);  // one speed for the fields between
    ap = __longlong_as_double((long long)lfb[NV - 1]);
  }
  // dv = L dU5 / 60 and Fc6 enter scaled by 60; the detector takes the 1/60
  constexpr double k60 = 1.0 / 60.0;
  double dv[NV];
  project<NV, DIR>(s, f.dU, dv);
  const double irho60 = s.irho * k60;
  unsigned weno = 0;
  if (hybrid == HYB_WENO_ONLY) {
    weno = (1u << NV) - 1u;
  } else if (hybrid != HYB_LINEAR_ONLY) {
    double vmax = fabs(dv[0]);
#pragma unroll
    for (int k = 1; k < NV; ++k) vmax = fmax(vmax, fabs(dv[k]));
    const double tm = vmax * irho60;
    const bool any = !(tm * tm < eps_thr);  // Eq.(30), (35)
    if (ANY) {
      weno = any ? 1u : 0u;
    } else if (hybrid == HYB_PER_FACE) {
      weno = any ? ((1u << NV) - 1u) : 0u;
    } else {
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        const double t = dv[k] * irho60;
        const double sig = t * t;
        if (!(sig < eps_thr)) weno |= 1u << k;
      }
    }
  }
  const double g = (am - a0) * dv[0], h = (ap - a0) * dv[NV - 1];
  const double S = g + h, D = s.c * (h - g);
#pragma unroll
  for (int i = 0; i < NV; ++i) F60[i] = f.F[i] + a0 * f.dU[i];
  F60[0] += S;
#pragma unroll
  for (int k = 0; k < DIM; ++k) F60[1 + k] += s.u[k] * S;
  F60[1 + DIR] += D;
  F60[NV - 1] += s.H * S;
  F60[NV - 1] += s.u[DIR] * D;
  // the state in the paper's units for a nonlinear correction (dead code,
  // removed by the compiler, where the caller drops it)
  st.s = s;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    st.a[k] = k == 0 ? am : (k == NV - 1 ? ap : a0);
    st.dv[k] = dv[k] * k60;
    st.Fc6[k] = f.F[k] * k60;
  }
  return weno;
}

// Linear-branch flux (times 60) of one face from six light records; returns
// whether some field's detector asks for the nonlinear flux.  `src.get(m,
// rec)` supplies stencil cell m = 0..5 (j-2 .. j+3).  SPLIT / HYB:
// compile-time splitting and switch modes, or -1 to read them from ph at run
// time.
template <int NV, int DIR, int SPLIT, int HYB, class Src>
__device__ __forceinline__ bool face_linear_l(const Src& src, const KPhys& ph, double eps_thr,
                                              const unsigned long long* lfb, double (&F60)[NV]) {
  FaceState<NV> st;
  return face_linear_st<NV, DIR, SPLIT, HYB, true>(src, ph, eps_thr, lfb, F60, st) != 0u;
}

// Index of a line position clamped to [-3, n+2] and mapped through the
// boundary rule; flip set for mirror ghosts.
__device__ __forceinline__ int ghost_clamped(int k, int n, int lo, int hi, bool& flip) {
  k = k < -3 ? -3 : (k > n + 2 ? n + 2 : k);
  return ghost_index(k, n, lo, hi, flip);
}

// Stencil accessor over six records held in registers.
template <int NV>
struct WinSrc {  // the owner's z window (registers)
  const LRec<NV>&w0, &w1, &w2, &w3, &w4, &w5;
  __device__ __forceinline__ void get(int m, LRec<NV>& r) const {
    r = m == 0 ? w0 : m == 1 ? w1 : m == 2 ? w2 : m == 3 ? w3 : m == 4 ? w4 : w5;
  }
};

// WENO-L2IS reconstruction at x_{j+1/2} from f_{j-2..j+2} (Eq.(5), (6),
// (11), (27), (28); optimal weights d = (0.4, 0.2, 0.3, 0.1)), the quotients
// through fast_rcp: the same formula as weno_l2is, a few ulp apart, with
// shorter dependency chains than correctly rounded division.  Every
// denominator is at least eps_w > 0 (the weight sum at least 1).  wts
// selects the comparison weights of Eq.(8) or Eq.(14)-(15) (lam unused).
__device__ __forceinline__ double weno_l2is_lr(double fm2, double fm1, double f0, double fp1,
                                               double fp2, double lam, double eps_w, int wts) {
  const double q0 = 0.5 * (f0 + fp1);
  const double q1 = 0.5 * (3.0 * f0 - fm1);
  const double q2 = (2.0 * f0 + 5.0 * fp1 - fp2) * (1.0 / 6.0);
  const double q3 = (2.0 * fm2 - 7.0 * fm1 + 11.0 * f0) * (1.0 / 6.0);
  const double d0 = fp1 - f0, d1 = f0 - fm1;
  const double b0 = d0 * d0, b1 = d1 * d1;
  const double s2a = f0 - 2.0 * fp1 + fp2, s2b = 3.0 * f0 - 4.0 * fp1 + fp2;
  const double s3a = fm2 - 2.0 * fm1 + f0, s3b = fm2 - 4.0 * fm1 + 3.0 * f0;
  const double b2 = (13.0 / 12.0) * s2a * s2a + 0.25 * s2b * s2b;
  const double b3 = (13.0 / 12.0) * s3a * s3a + 0.25 * s3b * s3b;
  const double t1 = (fp2 + fm2) - 4.0 * (fp1 + fm1) + 6.0 * f0;
  const double t2 = (fp2 - fm2) - 2.0 * (fp1 - fm1);
  const double tau5 = (13.0 / 12.0) * t1 * t1 + 0.25 * t2 * t2;
  const double e = fm1 - 2.0 * f0 + fp1;
  // one formula for the three weightings, the differences as selected
  // factors (no branch: both would hold their values in registers):
  // Eq.(28) d_k (1 + lam tau5 / (lam beta_k + E_k + eps)); Eq.(8) with lam
  // = 1 and E_k = 0; Eq.(14) with the numerator of the two-point stencils
  // multiplied by tau5 / (beta_01 + eps) of Eq.(15)
  const bool l2 = wts == W_L2IS;
  const double lv = l2 ? lam : 1.0;
  const double E01 = l2 ? e * e * (1.0 / 45.0) : 0.0;
  const double lt = lv * tau5;
  double n01 = lt;
  if (wts == W_IS_B01) {
    const double g = fm1 - fp1;
    n01 = tau5 * (tau5 * fast_rcp((13.0 / 12.0) * e * e + 0.25 * g * g + eps_w));
  }
  const double a0 = 0.4 * (1.0 + n01 * fast_rcp(lv * b0 + E01 + eps_w));
  const double a1 = 0.2 * (1.0 + n01 * fast_rcp(lv * b1 + E01 + eps_w));
  const double a2 = 0.3 * (1.0 + lt * fast_rcp(lv * b2 + eps_w));
  const double a3 = 0.1 * (1.0 + lt * fast_rcp(lv * b3 + eps_w));
  return (a0 * q0 + a1 * q1 + a2 * q2 + a3 * q3) * fast_rcp((a0 + a1) + (a2 + a3));
}

// The products of a shear row: the density's and component i's.
template <int NV>
__device__ __forceinline__ double dot2(const double (&r)[NV], const double (&x)[NV], int i) {
  double a = r[0] * x[0];  // the order of dot
  a += r[i] * x[i];
  return a;
}

// K: the field where it is known at compile time, else -1.  A shear row has
// two entries, so its products with zero are left out (they change no bit of a
// finite sum; a state that is not finite makes the acoustic fields NaN, and with
// them the face's whole flux, either way).
template <int NV, int DIR, int W, int K, class Src>
__device__ __forceinline__ double lean_field_row(const Src& src, const double (&r)[NV], const Roe<NV>& s,
                                                 double al, double dvk, const KPhys& ph) {
  constexpr bool SHEAR = K >= 2 && K < NV - 1;
  constexpr int comp = SHEAR ? (K - 2 < DIR ? K - 2 : K - 1) : 0;  // its momentum component
  double fp[6], fm[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    LRec<NV> cm;
    src.get(m, cm);
    double F[NV], un;
    lflux<NV, DIR>(cm, F, un);
    const double vv = SHEAR ? dot2<NV>(r, cm.U, 1 + comp) : dot<NV>(r, cm.U);
    const double gg = SHEAR ? dot2<NV>(r, F, 1 + comp) : dot<NV>(r, F);
    fp[m] = 0.5 * (gg + al * vv);
    fm[m] = 0.5 * (gg - al * vv);
  }
  const double t = dvk * s.irho;
  const double lam = ph.c_reg * (t * t);  // Eq.(32)
  const int wts = W >= 0 ? W : ph.weights;
  return weno_l2is_lr(fp[0], fp[1], fp[2], fp[3], fp[4], lam, ph.eps_w, wts) +
         weno_l2is_lr(fm[5], fm[4], fm[3], fm[2], fm[1], lam, ph.eps_w, wts);
}

template <int NV, int DIR, int K, int W, class Src>
__device__ __forceinline__ double lean_field(const Src& src, const Roe<NV>& s, double al, double dvk,
                                             const KPhys& ph) {
  double r[NV];
  left_row<NV, DIR, K>(s, r);
  return lean_field_row<NV, DIR, W, K>(src, r, s, al, dvk, ph);
}

// Row k of L for a field k known only at run time: each candidate row with
// the expressions of left_row<NV, DIR, k>, then selected (the same bits, no
// branch for lanes that take different fields).
template <int NV, int DIR>
__device__ __forceinline__ void left_row_rt(const Roe<NV>& s, int k, double (&r)[NV]) {
  constexpr int DIM = NV - 2;
  const double sg = k == 0 ? 1.0 : -1.0;
  double ac[NV], en[NV], sh[NV];
  ac[0] = 0.5 * (s.b2 + sg * s.u[DIR] * s.ic);
#pragma unroll
  for (int j = 0; j < DIM; ++j) ac[1 + j] = 0.5 * (-s.b1 * s.u[j] - (j == DIR ? sg * s.ic : 0.0));
  ac[NV - 1] = 0.5 * s.b1;
  en[0] = 1.0 - s.b2;
#pragma unroll
  for (int j = 0; j < DIM; ++j) en[1 + j] = s.b1 * s.u[j];
  en[NV - 1] = -s.b1;
  const int comp = (k - 2 < DIR) ? k - 2 : k - 1;  // shear field k-2: its momentum component
  double uc = 0.0;
#pragma unroll
  for (int j = 0; j < DIM; ++j) uc = j == comp ? s.u[j] : uc;
  sh[0] = -uc * s.ic;
#pragma unroll
  for (int j = 0; j < DIM; ++j) sh[1 + j] = (j == comp) ? s.ic : 0.0;
  sh[NV - 1] = 0.0;
  const bool acoustic = k == 0 || k == NV - 1;
#pragma unroll
  for (int i = 0; i < NV; ++i) r[i] = acoustic ? ac[i] : (k == 1 ? en[i] : sh[i]);
}

struct NoHook {
  __device__ __forceinline__ void operator()() const {}
};
// Nonlinear (WENO-L2IS) flux of one flagged face, field by field: for each
// field k in `mask`, the left eigenvector row L^k is formed, the six stencil
// cells are projected (Eq.(20)), split (Eq.(21)) and reconstructed
// (Eq.(22)-(23)); the other fields keep their linear flux.  The fields'
// fluxes are back-projected (Eq.(24)), and the correction is the difference
// from the linear face flux, R f - F60 / 60: where that is large and the WENO
// flux small (ambient cells next to a Mach 2000 jet), the sum of both keeps the
// rounding of the small one.  Only one row and twelve split values are live.
// W: the weighting (W_*) fixed at compile time, or -1 to read ph.weights.
// `early` runs before the last field (a kernel's loads for what follows).
template <int NV, int DIR, int W = -1, class Src, class Hook = NoHook>
__device__ __forceinline__ void lean_correction(const Src& src, unsigned mask, const FaceState<NV>& st,
                                                const double (&F60)[NV], const KPhys& ph,
                                                double (&dF)[NV], const Hook& early = Hook()) {
  double LF[NV], f[NV];
  project<NV, DIR>(st.s, st.Fc6, LF);
#define WL2_LF(K)                                                                                 \
  if constexpr (K < NV) {                                                                         \
    if constexpr (K == NV - 1) early();                                                           \
    f[K] = ((mask >> K) & 1u) ? lean_field<NV, DIR, K, W>(src, st.s, st.a[K], st.dv[K], ph)       \
                              : LF[K] + st.a[K] * st.dv[K];                                       \
  }
  WL2_LF(0) WL2_LF(1) WL2_LF(2) WL2_LF(3) WL2_LF(4)
#undef WL2_LF
  back_project<NV, DIR>(st.s, f, dF);
#pragma unroll
  for (int v = 0; v < NV; ++v) dF[v] -= F60[v] * (1.0 / 60.0);
}

// The six stencil cells of the face of cell (x, y, z) along DIR below it
// (side 0) or above it (side 1) as light records, with the boundary ghosts
// (all loads issued before any use).
template <int NV, int DIR>
__device__ __forceinline__ void face_stencil(const double* U, const KGrid& g, const KPhys& ph, int x,
                                             int y, int z, int side, LRec<NV> (&w)[6]) {
  // the face below the cell starts 3 cells below it, the face above 2 below
  const int c0 = (DIR == 0 ? x : DIR == 1 ? y : z) + (side ? -2 : -3);
  double u[6][NV];
  bool flip[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    const int k = ghost_clamped(c0 + m, g.n[DIR], g.bc_lo[DIR], g.bc_hi[DIR], flip[m]);
    int p[3] = {x, y, z};
    p[DIR] = k;
    const long long off = p[0] + (long long)p[1] * g.stride[1] + (long long)p[2] * g.stride[2];
#pragma unroll
    for (int v = 0; v < NV; ++v) u[m][v] = U[v * g.ncell + off];
  }
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    if (flip[m]) u[m][1 + DIR] = -u[m][1 + DIR];
    if (DIR == 0 && c0 + m < 0 && g.bc_lo[0] == BC_INFLOW)
      load_inflow<NV>(g, y + (long long)g.n[1] * z, u[m]);
    if (DIR == 1 && NV == 4 && (c0 + m < 0 || c0 + m >= g.n[1]) && is_yghost(g, c0 + m))
      load_yghost<NV>(g, x, c0 + m, u[m]);
    make_lrec<NV>(u[m], ph, w[m]);
  }
}

// Nonlinear correction of one face of cell (x, y, z) along DIR: side 0 is
// the face below the cell, side 1 the face above.  Returns the change of the
// face flux (WENO minus linear, Eq.(33) per field).
template <int NV, int DIR, int SPLIT, int HYB, int W = -1>
__device__ __forceinline__ void face_delta(const double* U, const KGrid& g, const KPhys& ph,
                                           const unsigned long long* lfb, int x, int y, int z,
                                           int side, double (&dF)[NV]) {
  // the six stencil cells, kept in registers for the linear flux and every
  // field's correction
  LRec<NV> w[6];
  face_stencil<NV, DIR>(U, g, ph, x, y, z, side, w);
  const WinSrc<NV> src{w[0], w[1], w[2], w[3], w[4], w[5]};
  double Flin[NV];
  FaceState<NV> st;
  const unsigned mask = face_linear_st<NV, DIR, SPLIT, HYB, false>(src, ph, ph.eps_thr[DIR], lfb, Flin, st);
  if (mask) {
    lean_correction<NV, DIR, W>(src, mask, st, Flin, ph, dF);
  } else {
#pragma unroll
    for (int v = 0; v < NV; ++v) dF[v] = 0.0;
  }
}

// The same change of flux computed by NV lanes of one wavefront, lane k of
// them (the lanes lane0 .. lane0 + NV - 1, all active here) taking field k:
// each forms the linear face and the correction of its own field, and the
// lanes exchange those to back-project them.  Every lane ends with the bits
// face_delta gives (the same operations per field, summed alike).
template <int NV, int DIR, int SPLIT, int HYB, int W = -1>
__device__ __forceinline__ void face_delta_field(const double* U, const KGrid& g, const KPhys& ph,
                                                 const unsigned long long* lfb, int x, int y, int z,
                                                 int side, int k, int lane0, double (&dF)[NV]) {
  LRec<NV> w[6];
  face_stencil<NV, DIR>(U, g, ph, x, y, z, side, w);
  const WinSrc<NV> src{w[0], w[1], w[2], w[3], w[4], w[5]};
  double Flin[NV];
  FaceState<NV> st;
  const unsigned mask = face_linear_st<NV, DIR, SPLIT, HYB, false>(src, ph, ph.eps_thr[DIR], lfb, Flin, st);
  double LF[NV];
  project<NV, DIR>(st.s, st.Fc6, LF);
  double al = st.a[0], dvk = st.dv[0], LFk = LF[0];
#pragma unroll
  for (int j = 1; j < NV; ++j) {
    al = j == k ? st.a[j] : al;
    dvk = j == k ? st.dv[j] : dvk;
    LFk = j == k ? LF[j] : LFk;
  }
  double mine = LFk + al * dvk;
  if ((mask >> k) & 1u) {
    double r[NV];
    left_row_rt<NV, DIR>(st.s, k, r);
    mine = lean_field_row<NV, DIR, W, -1>(src, r, st.s, al, dvk, ph);
  }
  double f[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) f[j] = __shfl(mine, lane0 + j, 64);
  if (mask) {
    back_project<NV, DIR>(st.s, f, dF);
#pragma unroll
    for (int v = 0; v < NV; ++v) dF[v] -= Flin[v] * (1.0 / 60.0);
  } else {
#pragma unroll
    for (int v = 0; v < NV; ++v) dF[v] = 0.0;
  }
}

// Nonlinear correction of one listed cell by one lane: the flagged faces in
// the fixed order x-, x+, y-, y+, z-, z+, +dF for the face below the cell and
// -dF for the face above.
template <int NV, int SPLIT, int HYB, int W = -1>
__device__ __forceinline__ void serial_correction(const double* U, const KGrid& g,
                                                  const KPhys& ph, const StepCtl* ctl, int x,
                                                  int y, int z, unsigned cm, double (&acc)[NV]) {
  constexpr int NF = 2 * (NV - 2);
#pragma unroll
  for (int v = 0; v < NV; ++v) acc[v] = 0.0;
  for (int f = 0; f < NF; ++f) {
    if (!((cm >> f) & 1u)) continue;
    const int dir = f >> 1, side = f & 1;
    double dF[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) dF[v] = 0.0;
    if (dir == 0) {
      face_delta<NV, 0, SPLIT, HYB, W>(U, g, ph, ctl->lf_bits[0], x, y, z, side, dF);
    } else if (dir == 1) {
      if constexpr (NV >= 4)
        face_delta<NV, (NV >= 4 ? 1 : 0), SPLIT, HYB, W>(U, g, ph, ctl->lf_bits[1], x, y, z, side, dF);
    } else {
      if constexpr (NV >= 5)
        face_delta<NV, (NV >= 5 ? 2 : 0), SPLIT, HYB, W>(U, g, ph, ctl->lf_bits[2], x, y, z, side, dF);
    }
    const double sg = side ? -1.0 : 1.0;
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] += sg * dF[v];
  }
}

// Nonlinear correction of one listed cell, computed by a group of GRP lanes
// of one wavefront: lane f of the group takes face f = 2 dir + side (x-, x+,
// y-, y+, z-, z+) if the mask flags it, and every lane of the group gets the
// sum of +-dF over the flagged faces in that fixed order (the face below the
// cell adds, the face above subtracts): the same bits as serial_correction,
// with one face of latency instead of six (for short lists; a long list
// keeps every lane busy with one cell each).
template <int NV, int GRP, int SPLIT, int HYB, int W = -1>
__device__ __forceinline__ void grouped_correction(const double* U, const KGrid& g,
                                                   const KPhys& ph, const StepCtl* ctl, int x,
                                                   int y, int z, unsigned cm, double (&acc)[NV]) {
  constexpr int NF = 2 * (NV - 2);
  static_assert(NF <= GRP && (64 % GRP) == 0, "one lane per face, groups inside a wavefront");
  const int lane = threadIdx.x & 63;
  const int f = lane % GRP;
  const int lane0 = lane - f;
  double dF[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) dF[v] = 0.0;
  if (f < NF && ((cm >> f) & 1u)) {
    const int dir = f >> 1, side = f & 1;
    if (dir == 0) {
      face_delta<NV, 0, SPLIT, HYB, W>(U, g, ph, ctl->lf_bits[0], x, y, z, side, dF);
    } else if (dir == 1) {
      if constexpr (NV >= 4)
        face_delta<NV, (NV >= 4 ? 1 : 0), SPLIT, HYB, W>(U, g, ph, ctl->lf_bits[1], x, y, z, side, dF);
    } else {
      if constexpr (NV >= 5)
        face_delta<NV, (NV >= 5 ? 2 : 0), SPLIT, HYB, W>(U, g, ph, ctl->lf_bits[2], x, y, z, side, dF);
    }
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) acc[v] = 0.0;
#pragma unroll
  for (int ff = 0; ff < NF; ++ff) {
    double d[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) d[v] = __shfl(dF[v], lane0 + ff, 64);
    if ((cm >> ff) & 1u) {
      const double sg = (ff & 1) ? -1.0 : 1.0;
#pragma unroll
      for (int v = 0; v < NV; ++v) acc[v] += sg * d[v];
    }
  }
}

}  // namespace wl2
