// Device code of libdgmoist: the pointwise implicit-condensation split, the
// pointwise state/flux/source evaluation and the fused right-hand-side kernel.
//
// Precision: the split (Newton on the implicit condensation system of
// Section 2.2), the reconstruction of full densities, p' = p - p_bar and
// rho e from the stored perturbations are always FP64.  Fluxes, the
// sum-factorised volume contraction, face fluxes, sources and the stage
// update run in the state's precision R (double, or float in FP32-bulk mode)
// with accumulation in R.
#pragma once
#include "dg_common.h"

namespace dgm {

// The constant address space (read-only global memory; scalar loads) in the
// device pass.
#if defined(__HIP_DEVICE_COMPILE__)
#define DGM_AS_CONST __attribute__((address_space(4)))
#else
#define DGM_AS_CONST
#endif

template <int D, int RAIN>
struct Vars {
  static constexpr int NV = 3 + D + RAIN;
  static constexpr int RD = 0, RM = 1, RR = 2, M0 = 2 + RAIN, E = NV - 1;
};

// Threads per block: 256 in FP32; 128 in FP64, where the LDS tiles are twice
// as large and 256-thread blocks would leave room for only two per CU.
template <typename R>
constexpr int block_threads() { return sizeof(R) == 4 ? 256 : 128; }

template <int K, int D, int BT = 256>
struct Shape {
  static constexpr int P1 = K + 1;
  static constexpr int NP = (D == 2) ? P1 * P1 : P1 * P1 * P1;
  static constexpr int EPB = (BT / NP) > 0 ? BT / NP : 1;   // elements per block
  static constexpr int NT = EPB * NP;                          // threads per block
};

// ---------------------------------------------------------------------------
// per-variable device arrays through buffer resources
// ---------------------------------------------------------------------------
// One 128-bit descriptor (base address, byte size, raw 32-bit data format)
// per array, built with scalar instructions; accesses take a 32-bit byte
// offset, so no 64-bit address arithmetic per load, and the hardware drops
// accesses past the end (reads return 0).  Array byte sizes stay below 4 GiB
// (the handle limits its node count accordingly).
constexpr int kRawBufferWord3 = 0x00020000;

template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const T* base, unsigned n) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)(n * (unsigned)sizeof(T)), kRawBufferWord3);
}

__device__ __forceinline__ float buf_load(__amdgpu_buffer_rsrc_t r, unsigned i, float*) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, i * 4u, 0, 0));
}
__device__ __forceinline__ double buf_load(__amdgpu_buffer_rsrc_t r, unsigned i, double*) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, i * 8u, 0, 0));
}
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, unsigned i, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, i * 4u, 0, 0);
}
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, unsigned i, double v) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, i * 8u, 0, 0);
}

// element i of variable v of an SoA state (v-major, n nodes per variable)
template <typename T>
__device__ __forceinline__ T ld(const T* base, unsigned n, int v, unsigned i) {
  return buf_load(buf_rsrc(base + (size_t)v * n, n), i, (T*)nullptr);
}
template <typename T>
__device__ __forceinline__ void st(T* base, unsigned n, int v, unsigned i, T x) {
  buf_store(buf_rsrc(base + (size_t)v * n, n), i, x);
}

// Value i of an FP64 array of one value per node (T, rho_vs) beside a state in
// R.  An FP32 handle holds up to 2^30 nodes, and from 2^29 on such an array
// outgrows a 32-bit byte offset: there it is addressed by pointer (one 64-bit
// add per access, in bounds by the caller).
template <typename R>
__device__ __forceinline__ double ld_f64(const double* base, unsigned n, unsigned i) {
  if constexpr (sizeof(R) == 4) return base[i];
  else return ld(base, n, 0, i);
}
template <typename R>
__device__ __forceinline__ void st_f64(double* base, unsigned n, unsigned i, double x) {
  if constexpr (sizeof(R) == 4) base[i] = x;
  else st(base, n, 0, i, x);
}

// ---------------------------------------------------------------------------
// saturation vapour density and the split (FP64)
// ---------------------------------------------------------------------------
// FP64 reciprocal: hardware estimate refined by two Newton steps
__device__ __forceinline__ double rcp64(double v) {
  double r = __builtin_amdgcn_rcp(v);
  r = fma(fma(-v, r, 1.0), r, r);
  r = fma(fma(-v, r, 1.0), r, r);
  return r;
}

// rho_vs(T) = e_s(T) / (R_v T) with the Clausius-Clapeyron e_s of Section 2.1,
// written as one exponential: C0 exp((a - 1) ln(T/T_ref) + b (1/T_ref - 1/T)).
// The logarithm is 2 atanh((m - 1)/(m + 1)) of the mantissa m in [1/sqrt 2,
// sqrt 2) (its Taylor series to z^10, remainder 2e-19), the exponential a Taylor
// polynomial on |r| <= (ln 2)/2 (to r^13, remainder 4e-18).  What counts is the
// absolute error of the exponent (up to 30 in size), so a logarithm to 3e-16
// absolute serves; the library's, correct to the last bit near 1, and its
// exponential took 100 of this function's 155 VALU instructions (65 now).
// Against 64-bit mantissas over T = 150 .. 600 K the largest relative error is
// 7.4e-15 (library functions 7.1e-15), the rms 1.39e-15 (1.40e-15).  Two
// cold splits and a right-hand side on 50 x 42 x 26 Q3 in FP32: 175 -> 160 us.
__device__ __forceinline__ double rho_vs(const KArgs& a, double T, double iT) {
  const double x = T * a.inv_Tref;
  double m = __builtin_amdgcn_frexp_mant(x);
  int e = __builtin_amdgcn_frexp_exp(x);
  const bool low = m < 0.70710678118654752;
  m = low ? m + m : m;
  e = low ? e - 1 : e;
  const double s = (m - 1.0) * rcp64(m + 1.0), z = s * s;
  double p = 2.0 / 21;
#pragma unroll
  for (int k = 19; k >= 3; k -= 2) p = fma(p, z, 2.0 / k);
  const double l = fma((double)e, 0.69314718055994531, fma(s * z, p, s + s));
  const double u = fmax(fma(a.am1, l, a.b * (a.inv_Tref - iT)), -745.2);   // (below, exp is 0)
  const double n = rint(u * 1.4426950408889634);
  double r = fma(n, -0.69314718055994531, u);
  r = fma(n, -2.3190468138462996e-17, r);
  double q = 1.0 / 6227020800.0;   // 1/13!
  const double f[13] = {1.0 / 479001600, 1.0 / 39916800, 1.0 / 3628800, 1.0 / 362880, 1.0 / 40320, 1.0 / 5040, 1.0 / 720,
                  1.0 / 120, 1.0 / 24, 1.0 / 6, 0.5, 1.0, 1.0};
#pragma unroll
  for (int k = 0; k < 13; ++k) q = fma(q, r, f[k]);
  return T > 0.0 ? a.C0 * ldexp(q, (int)n) : __builtin_nan("");
}
__device__ __forceinline__ double rho_vs(const KArgs& a, double T) { return rho_vs(a, T, rcp64(T)); }

struct SplitOut {
  double T;     // temperature
  double rvs;   // rho_vs(T); rho_v = min(rvs, rho_m)
  int iters;    // Newton iterations (0 when unsaturated)
  int bad;      // 1: no valid temperature, 2: iteration cap reached
};

// rho_vs near an anchor temperature T0 where r0 = rho_vs(T0) is known:
//   rho_vs(T) = r0 exp(phi(T) - phi(T0)),
//   phi(T) - phi(T0) = (a - 1) log(1 + x) + b x / (T0 (1 + x)),  x = (T - T0)/T0,
// with log(1 + x), 1/(1 + x) and exp(.) - 1 summed as Taylor series.  For
// |x| <= kAnchorX the truncation errors are below 1e-19 relative (|x|^8/8,
// |x|^8 and |dphi|^11/11! with |dphi| < 0.09 for T0 >= 200 K).
constexpr double kAnchorX = 2.0e-3;

struct Anchor {
  double T0, r0, inv0;
};

__device__ __forceinline__ Anchor make_anchor(const KArgs& a, double T) {
  Anchor A;
  A.T0 = T;
  A.inv0 = rcp64(T);
  A.r0 = rho_vs(a, T, A.inv0);
  return A;
}

__device__ __forceinline__ bool in_anchor(const Anchor& A, double T) {
  return fabs(T - A.T0) <= kAnchorX * A.T0;
}

// Between two stages T moves by far less than the anchor range, and for
// |x| <= kShortX shorter series suffice (anchors lie above 150 K, so
// b / T0 < 46): log(1 + x) to x^4 (error |x|^5/5 < 3e-21), 1/(1 + x) to x^3
// (error x^4 = 1e-16, entering d multiplied by b x / T0 < 5e-3) and
// exp(d) - 1 to d^5 (|d| < 5.2e-3, error d^6/720 < 3e-17).  The choice is
// made per wavefront.
constexpr double kShortX = 1.0e-4;

// rho_vs(T) and d rho_vs / dT from the anchor
__device__ __forceinline__ double rvs_near(const KArgs& a, const Anchor& A, double T, double* drvs) {
  const double x = (T - A.T0) * A.inv0;
  double l, q, e;
  if (__all(x == 0.0)) {
    // at the anchor itself (the first step of a warm-started solve): the
    // series below give exactly these values for x = 0
    *drvs = A.r0 * (a.am1 + a.b * A.inv0) * A.inv0;
    return A.r0;
  }
  if (__all(fabs(x) <= kShortX)) {
    l = x * (1.0 + x * (-0.5 + x * (1.0 / 3.0 - x * 0.25)));
    q = 1.0 + x * (-1.0 + x * (1.0 - x));
    const double d = a.am1 * l + a.b * A.inv0 * x * q;
    e = d * (1.0 + d * (1.0 / 2 + d * (1.0 / 6 + d * (1.0 / 24 + d * (1.0 / 120)))));
  } else {
    l = x * (1.0 + x * (-0.5 + x * (1.0 / 3.0 + x * (-0.25 + x * (0.2 + x * (-1.0 / 6.0 + x * (1.0 / 7.0)))))));
    q = 1.0 + x * (-1.0 + x * (1.0 + x * (-1.0 + x * (1.0 + x * (-1.0 + x * (1.0 - x))))));
    const double d = a.am1 * l + a.b * A.inv0 * x * q;
    e = d * (1.0 + d * (1.0 / 2 + d * (1.0 / 6 + d * (1.0 / 24 + d * (1.0 / 120 + d * (1.0 / 720 +
        d * (1.0 / 5040 + d * (1.0 / 40320 + d * (1.0 / 362880 + d * (1.0 / 3628800))))))))));
  }
  const double r = A.r0 + A.r0 * e;
  const double invT = A.inv0 * q;
  *drvs = r * (a.am1 + a.b * invT) * invT;
  return r;
}

// Implicit condensation (Section 2.2): find T with
//   rho e = (c_vd rd + c_vv rv + c_l (rm - rv + rr)) (T - T_ref) + rv (L_ref - R_v T_ref),
//   rv = min(rho_vs(T), rm).
// The map T -> rho e is strictly increasing, so the root is unique.  Each
// branch gives a candidate and an exact test:
//   unsaturated: T = Tu (all water as vapour), valid iff rm <= rho_vs(Tu);
//   saturated:   the root Ts of f(T) = rho e(T, rv = rho_vs(T)) - rho e,
//                valid iff rho_vs(Ts) <= rm (then Ts is the unique root).
// `sat_first` names the branch to try first (with a warm start, the branch
// that held before), so a node normally evaluates one branch.  On the
// saturated branch f is increasing and convex; Newton evaluates rho_vs by
// series around an anchor that is re-based when an iterate leaves its range.
// The Newton step uses the hardware reciprocal of f' (relative error far
// below the step's own size, so convergence stays quadratic).  Stopping:
// |dT| <= rtol T, or, above 150 K, the quadratic-convergence bound: after a
// step dT the error is at most M dT^2 with M = max |f''| / (2 min f').  With
// f' >= rho_vs' L_eff and f'' <= rho_vs'' L_eff (the c_vv - c_l term is below
// 2e-3 of it), M <= (q + q'/q)/2 + 2e-3 with q = d ln rho_vs / dT, which is
// 0.15 K^-1 at 150 K and falls with T; M = 0.25 K^-1 is used, so
// |dT| <= sqrt(rtol T / M) already leaves an error below rtol T.
// If `A` holds a valid anchor (A.T0 > 0) it is used and updated in place.
struct NewtonOut {
  double T, rvs;
  int iters;
  int state;   // 0 converged, 1 root lies below Tu (not saturated), 2 iteration cap
};

__device__ __forceinline__ NewtonOut newton_sat(const KArgs& a, double Cu, double rm, double re,
                                                double Tu, double lo, double T, Anchor& A) {
  const double dc = a.cvv - a.cl;
  if (!(A.T0 > 0.0) || !in_anchor(A, T)) A = make_anchor(a, T);
  // |dT| <= tol with tol = rtol T, or above 150 K max(rtol T, 2 sqrt(rtol T)),
  // compared as squares
  const double tol_lin = a.rtol * T;
  const double tol2 = T > 150.0 ? fmax(tol_lin * tol_lin, 4.0 * tol_lin) : tol_lin * tol_lin;
  NewtonOut o;
  o.state = 2;
  double rvs = 0.0;
  int it = 0;
  while (it < a.maxit) {
    if (!in_anchor(A, T)) A = make_anchor(a, T);
    double drvs;
    rvs = rvs_near(a, A, T, &drvs);
    const double Cv = Cu + dc * (rvs - rm);
    const double Tm = T - a.Tref;
    const double f = Cv * Tm + rvs * a.Lp - re;
    const double fp = Cv + drvs * (dc * Tm + a.Lp);
    const double dT = -f * __builtin_amdgcn_rcp(fp);
    ++it;
    if (dT * dT <= tol2) {
      T += dT;
      rvs += drvs * dT;          // first order is exact to rounding for this step size
      o.state = 0;
      break;
    }
    double Tn = T + dT;
    if (!(Tn > lo)) {
      // f is convex: from the right of the root Newton never overshoots, so a
      // step below the bound means the saturated root lies below Tu
      if (f > 0.0 && lo == Tu) { o.state = 1; break; }
      Tn = 0.5 * (T + lo);
    }
    T = Tn;
  }
  o.T = T;
  o.rvs = rvs;
  o.iters = it;
  return o;
}

__device__ __forceinline__ SplitOut split_point_anchor(const KArgs& a, double rd, double rm, double rr,
                                                       double re, double guess, Anchor& A,
                                                       bool sat_first = false) {
  SplitOut o;
  o.iters = 0;
  o.bad = 0;
  const double Cu = a.cvd * rd + a.cvv * rm + a.cl * rr;
  const double Tu = a.Tref + (re - rm * a.Lp) * rcp64(Cu);
  if (!isfinite(Tu) || !(Cu > 0.0)) {
    o.T = __builtin_nan(""); o.rvs = rm; o.bad = 1;
    return o;
  }
  // unsaturated test
  bool unsat = false;
  double rTu = 0.0;
  if (!sat_first && Tu > 0.0) {
    double dr;
    rTu = (A.T0 > 0.0 && in_anchor(A, Tu)) ? rvs_near(a, A, Tu, &dr) : rho_vs(a, Tu);
    unsat = rm <= rTu;
  }
  if (!unsat) {
    // saturated branch: Newton from the warm start if it lies above the
    // branch's lower bound max(Tu, 50 K)
    double lo = Tu;
    if (!(Tu > 50.0)) {
      const double r = rho_vs(a, 50.0);
      const double f = (Cu + (a.cvv - a.cl) * (r - rm)) * (50.0 - a.Tref) + r * a.Lp - re;
      if (!(f < 0.0)) { o.T = __builtin_nan(""); o.rvs = rm; o.bad = 1; return o; }
      lo = 50.0;
    }
    const double T0 = (guess > lo && guess < 600.0) ? guess : lo;
    const NewtonOut n = newton_sat(a, Cu, rm, re, Tu, lo, T0, A);
    o.iters = n.iters;
    if (n.state == 2) { o.T = n.T; o.rvs = rho_vs(a, n.T); o.bad = 2; return o; }
    if (n.state == 0 && (n.rvs <= rm || !(Tu > 0.0))) { o.T = n.T; o.rvs = n.rvs; return o; }
    // the saturated root is not a solution: the air is unsaturated
    if (!sat_first) { o.T = Tu; o.rvs = rm; return o; }   // ties at the branch point
    rTu = rho_vs(a, Tu);
  }
  o.T = Tu;
  o.rvs = rTu;
  return o;
}

__device__ __forceinline__ SplitOut split_point(const KArgs& a, double rd, double rm, double rr,
                                                double re, double guess) {
  Anchor A;
  A.T0 = 0.0; A.r0 = 0.0; A.inv0 = 0.0;
  return split_point_anchor(a, rd, rm, rr, re, guess, A);
}

// ---------------------------------------------------------------------------
// the split near a point of the saturation curve, without iterations
// ---------------------------------------------------------------------------
// With (T0, r0 = rho_vs(T0)) known and y = (T - T0)/T0, rho_vs is
//   r0 (1 + Q y + P2 y^2 + P3 y^3 + P4 y^4),
// the Taylor series of exp(phi), phi = (a - 1) ln T - b/T, with
// Q = T0 phi'(T0) = a - 1 + b/T0.  For |Q y| <= kNearQ the truncation,
// |Q y|^5/120 < 3e-16, is below rounding.  On the saturated branch
//   f(y) = Cs (T - T_ref) + rho_vs (dc (T - T_ref) + L_p) - rho e,
//   Cs = c_vd rd + c_l (rm + rr), dc = c_vv - c_l,
// is then a quartic f0 + f1 y + ... + f4 y^4; its root is -f0/f1 corrected by
// one quadratic term and one Newton step on the quartic, whose relative
// error is of the order (Q y)^4 (1.6e-11 of a change of at most 0.1 K).  The
// unsaturated candidate is the closed form T_u.  The caller names the branch
// (`sat`); `ok` says that the candidate passed that branch's own exact test
// (the root is unique, so it is then the solution).  Everything else (branch
// changes, large changes, invalid states) is left to split_point_anchor.
// Bound by VALU issue: the warm solve replaces two or three iterations (one
// rvs_near each) of every stage; with the cold solve below, steps of five
// 3D Q3 FP32 calls 6.20 -> 5.82 ms, the 64-member 2D ensemble 3.28 -> 3.01 ms.
constexpr double kNearQ = 2.0e-3;
constexpr int kEstIters = 8;   // single-precision steps of split_scratch at most

struct NearOut {
  double T, rvs;
  bool ok;
};

__device__ __forceinline__ NearOut split_near(const KArgs& a, double rd, double rm, double rr, double re,
                                              double T0, double r0, double inv0, bool sat) {
  NearOut o;
  const double dc = a.cvv - a.cl;
  const double Cs = fma(a.cvd, rd, a.cl * (rm + rr));
  const double Cu = fma(dc, rm, Cs);
  const double beta = a.b * inv0;
  const double Q = a.am1 + beta;
  // T0^n times the n-th derivative of phi, n = 2, 3, 4
  const double c2 = -(Q + beta), c3 = 2.0 * (Q + 2.0 * beta), c4 = -6.0 * (Q + 3.0 * beta);
  const double Q2 = Q * Q;
  const double P2 = 0.5 * (Q2 + c2);
  const double P3 = (1.0 / 6.0) * fma(Q, Q2 + 3.0 * c2, c3);
  const double P4 = (1.0 / 24.0) * (fma(Q2, Q2 + 6.0 * c2, fma(4.0 * Q, c3, fma(3.0 * c2, c2, c4))));
  double y;
  if (sat) {
    const double Tm = T0 - a.Tref;
    const double g = fma(dc, Tm, a.Lp);
    const double rg = r0 * g, rt = r0 * dc * T0;
    const double f0 = fma(Cs, Tm, rg - re);
    const double f1 = fma(Cs, T0, fma(rg, Q, rt));
    double i1 = __builtin_amdgcn_rcp(f1);
    i1 = fma(fma(-f1, i1, 1.0), i1, i1);
    const double y0 = -f0 * i1;
    const double k2 = fma(rg, P2, rt * Q) * i1;
    const double k3 = fma(rg, P3, rt * P2) * i1;
    const double k4 = fma(rg, P4, rt * P3) * i1;
    const double y1 = fma(-k2 * y0, y0, y0);
    const double p = fma(y1 * y1, fma(y1, fma(y1, k4, k3), k2), y1 - y0);
    y = fma(-p, fma(-2.0 * k2, y1, 1.0), y1);
  } else {
    const double Tu = a.Tref + (re - rm * a.Lp) * rcp64(Cu);
    y = (Tu - T0) * inv0;
  }
  const double e = y * fma(y, fma(y, fma(y, P4, P3), P2), Q);
  o.T = fma(y, T0, T0);
  o.rvs = fma(r0, e, r0);
  const bool branch = sat ? o.rvs <= rm : rm <= o.rvs;
  o.ok = branch && fabs(Q * y) <= kNearQ && Cu > 0.0 && T0 > 150.0 && T0 < 600.0 && r0 > 0.0;
  return o;
}

// A larger change (up to kAnchorX): the quartic's root is within 1e-6 K; one
// Newton step with rho_vs and its slope from the anchored series completes it
// (error below 0.25 K^-1 dT^2, see newton_sat).  The series are those of
// rvs_near for |x| <= kAnchorX, without the choice per wavefront.
__device__ __forceinline__ NearOut split_mid(const KArgs& a, double rd, double rm, double rr, double re,
                                             double T0, double r0, double inv0, bool sat, double Tn) {
  NearOut o;
  const double x = (Tn - T0) * inv0;
  const double l = x * (1.0 + x * (-0.5 + x * (1.0 / 3.0 + x * (-0.25 + x * (0.2 + x * (-1.0 / 6.0 + x * (1.0 / 7.0)))))));
  const double q = 1.0 + x * (-1.0 + x * (1.0 + x * (-1.0 + x * (1.0 + x * (-1.0 + x * (1.0 - x))))));
  const double d = a.am1 * l + a.b * inv0 * x * q;
  const double e = d * (1.0 + d * (1.0 / 2 + d * (1.0 / 6 + d * (1.0 / 24 + d * (1.0 / 120 + d * (1.0 / 720 +
      d * (1.0 / 5040 + d * (1.0 / 40320 + d * (1.0 / 362880 + d * (1.0 / 3628800))))))))));
  o.T = Tn;
  o.rvs = r0 + r0 * e;
  bool small = true;
  if (sat) {
    const double dc = a.cvv - a.cl, iT = inv0 * q;
    const double dr = o.rvs * (a.am1 + a.b * iT) * iT;
    const double Cv = fma(a.cvd, rd, a.cl * (rm + rr)) + dc * o.rvs;
    const double Tm = Tn - a.Tref;
    const double dT = -(Cv * Tm + o.rvs * a.Lp - re) * rcp64(Cv + dr * (dc * Tm + a.Lp));
    o.T += dT;
    o.rvs += dr * dT;
    small = dT * dT <= 4.0e-14 * Tn;
  }
  const bool branch = sat ? o.rvs <= rm : rm <= o.rvs;
  o.ok = branch && small && fabs(x) <= kAnchorX && T0 > 150.0 && T0 < 600.0 && r0 > 0.0;
  return o;
}

// The split warm-started at the node's previous (T, rho_vs(T)); the branch that
// held there before is tried first.  Without the closed form (KArgs::closed) 2D
// kernels skip it (two steps on 350 x 175 Q2 in FP32, cap 8: 241 -> 218 us); in 3D
// the quartic is solved and thrown away, as the branch around it costs registers
// that the FP64 kernels do not have (Gauss basis with rain, 32 x 31 x 16 Q3, two
// steps: 863 -> 900 us).
template <int D>
__device__ __forceinline__ SplitOut split_warm(const KArgs& a, double rd, double rm, double rr, double re, double T,
                                               double rvs) {
  const double inv = rcp64(T);
  const bool sat = rvs < rm;
  SplitOut o;
  o.iters = sat ? 1 : 0;
  o.bad = 0;
  bool ok = false;
  if (D == 3 || a.closed) {
    NearOut n = split_near(a, rd, rm, rr, re, T, rvs, inv, sat);
    const bool pos = fma(a.cvd, rd, a.cl * (rm + rr)) + (a.cvv - a.cl) * rm > 0.0;
    if (!n.ok && pos && a.closed) {
      n = split_mid(a, rd, rm, rr, re, T, rvs, inv, sat, n.T);
      o.iters = sat ? 2 : 0;
    }
    ok = n.ok && a.closed;
    o.T = n.T;
    o.rvs = n.rvs;
  }
  if (!ok) {
    Anchor A;
    A.T0 = 0.0; A.r0 = 0.0; A.inv0 = 0.0;
    if (T > 150.0 && T < 600.0 && rvs > 0.0) {
      A.T0 = T; A.r0 = rvs; A.inv0 = inv;
    }
    o = split_point_anchor(a, rd, rm, rr, re, T, A, sat);
  }
  return o;
}

// rho_vs in single precision (hardware exp2/log2; relative error below 1e-5)
// and d ln rho_vs / dT
__device__ __forceinline__ float rho_vs_est(const KArgs& a, float T, float* q) {
  const float iT = __builtin_amdgcn_rcpf(T);
  const float l = __builtin_amdgcn_logf(T * (float)a.inv_Tref);
  *q = ((float)a.am1 + (float)a.b * iT) * iT;
  return (float)a.C0 *
         __builtin_amdgcn_exp2f((float)a.am1 * l + (float)(a.b * 1.4426950408889634) * ((float)a.inv_Tref - iT));
}

// The split from scratch (no rho_vs known nearby).  Single precision finds the
// branch and, on the saturated one, the temperature to about 1e-4 K (Newton
// from the guess if it lies above T_u, else from T_u); one FP64 rho_vs there
// is the anchor of split_near, which gives the FP64 result.  Within 1e-4 of
// the branch point the anchor is T_u itself and the FP64 value decides.  The
// returned rho_vs(T) comes from a fresh evaluation at most 0.03 K away (the
// estimate's error), so it can anchor later splits.  `iters` counts the
// estimate's steps and the FP64 solve; a cap (newton_maxit) below what this
// may use, or a tolerance below what it gives, takes the general path.
// FP64 iterations throughout took 970-1100 VALU instructions per wavefront
// (three or four exp/log anchors) and kept the VALU 75-100 % busy; two cold
// splits and a right-hand side on 50 x 42 x 26 Q3 in FP32: 272 -> 177 us.

__device__ __forceinline__ SplitOut split_scratch(const KArgs& a, double rd, double rm, double rr, double re,
                                                  double guess) {
  SplitOut o;
  bool ok = false;
  if (a.closed) {
    const double Cs = fma(a.cvd, rd, a.cl * (rm + rr));
    const double Cu = fma(a.cvv - a.cl, rm, Cs);
    const double Tu = a.Tref + (re - rm * a.Lp) * rcp64(Cu);
    float q;
    bool sat = (float)rm > 1.0001f * rho_vs_est(a, (float)Tu, &q);
    double T1 = Tu;
    int it = 0;
    if (sat) {
      const float dc = (float)(a.cvv - a.cl), tref = (float)a.Tref, Lp = (float)a.Lp, cs = (float)Cs, ref = (float)re;
      float T = (float)(guess > Tu && guess < 600.0 ? guess : Tu);
      float dT;
      do {
        const float r = rho_vs_est(a, T, &q);
        const float g = dc * (T - tref) + Lp;
        dT = (cs * (T - tref) + (r * g - ref)) * __builtin_amdgcn_rcpf(cs + r * (q * g + dc));
        T -= dT;
        ++it;
      } while (fabsf(dT) > 0.02f && it < kEstIters);
      T1 = (double)T;
    }
    const double i1 = rcp64(T1), r0 = rho_vs(a, T1, i1);
    sat = sat || rm > r0;
    const NearOut n = split_near(a, rd, rm, rr, re, T1, r0, i1, sat);
    ok = n.ok;
    o.T = n.T;
    o.rvs = n.rvs;
    o.iters = sat ? it + 1 : 0;
    o.bad = 0;
  }
  if (!ok) {
    o = split_point(a, rd, rm, rr, re, guess);
    if (o.iters > 0 && o.bad == 0) o.rvs = rho_vs(a, o.T);
  }
  return o;
}

// Status words: only exceptional events touch global memory.  `seen` is the
// block's stored iteration maximum as it stood when the kernel began (a uniform
// load issued with the first ones, not a round trip at the end of every wave);
// a wave that exceeds it forms its maximum and checks the current value before
// the atomic.  Non-converged or invalid states are rare.
__device__ __forceinline__ unsigned* stat_slot(const KArgs& a) {
  return a.stats + kStatStride * (1 + (blockIdx.x & (kStatSlots - 1)));
}

__device__ __forceinline__ int wave_max(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return v;
}

__device__ __forceinline__ int stats_seen(const KArgs& a) {
  return (int)*(const unsigned DGM_AS_CONST*)(unsigned long long)stat_slot(a);
}

__device__ __forceinline__ void record_stats(const KArgs& a, int seen, int iters, int bad) {
  if (__any(iters > seen)) {
    const int m = wave_max(iters);
    unsigned* const w = stat_slot(a);
    if ((threadIdx.x & 63) == 0 &&
        (unsigned)m > __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(w, (unsigned)m);
  }
  if (__any(bad != 0)) {
    if (bad == 2) atomicAdd(&a.stats[1], 1u);
    if (bad == 1) atomicOr(&a.stats[2], 1u);
  }
}

// ---------------------------------------------------------------------------
// pointwise state, fluxes, wave speed and sources
// ---------------------------------------------------------------------------
// reciprocal and fractional power in the bulk precision: hardware
// reciprocal/log2/exp2 in FP32 (about 1 ulp), refined or library forms in FP64
__device__ __forceinline__ float inv_b(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double inv_b(double x) { return rcp64(x); }
__device__ __forceinline__ float pow_b(float x, float p) {
  return __builtin_amdgcn_exp2f(p * __builtin_amdgcn_logf(x));
}
__device__ __forceinline__ double pow_b(double x, double p) { return pow(x, p); }
// x^(3/16), x^(1/2) and x^(7/8) of the Kessler terms: in FP64 from square
// roots, x^(1/8) x^(1/16) and x / x^(1/8) (two library pow calls were 40 % of
// the FP64 stage kernel's instructions)
__device__ __forceinline__ void kessler_pow(float x, float& p316, float& p12, float& p78) {
  p316 = pow_b(x, 0.1875f);
  p12 = sqrt(x);
  p78 = pow_b(x, 0.875f);
}
__device__ __forceinline__ void kessler_pow(double x, double& p316, double& p12, double& p78) {
  p12 = sqrt(x);
  const double p18 = sqrt(sqrt(p12));
  p316 = p18 * sqrt(p18);
  p78 = x / p18;
}

template <typename R, int D, int RAIN>
struct Pt {
  R m[D], u[D];
  R rd, rm, rr;     // full densities
  R rho;            // total density
  R H;              // E + p_bar + p'
  R pp;             // p'
  R cm;             // moist sound speed
  R vr;             // terminal rain speed
  R rrvr;           // rho_r v_r
  R rain_e;         // (c_l (T - T_ref) + u.u/2) rho_r v_r
  R rc, dvs, Tm;    // rho_c, rho_vs(T) - rho_v, T - T_ref (rain only)
};

// Full state from the perturbation Uq, the temperature T, the vapour density
// rho_v and the background (rho_d, rho_m, rho_r, p, E + p) at the point; rho_vs
// enters only the evaporation source.  The reconstruction is FP64.
template <typename R, int D, int RAIN>
__device__ __forceinline__ void eval_core(const KArgs& a, const R* Uq, double T, double rv, double rvs,
                                          double bd, double bm, double br, double bp, double bEp,
                                          Pt<R, D, RAIN>& q) {
  using V = Vars<D, RAIN>;
  const double rd = bd + (double)Uq[V::RD];
  const double rm = bm + (double)Uq[V::RM];
  const double rr = RAIN ? br + (double)Uq[V::RR] : 0.0;
  const double rc = rm - rv;
  const double gasR = rd * a.Rd + rv * a.Rv;
  const double p = gasR * T;
  const double ppd = p - bp;
  const double rho = rd + rm + rr;
  const double Cv = a.cvd * rd + a.cvv * rv + a.cl * (rc + rr);
  q.rd = (R)rd; q.rm = (R)rm; q.rr = (R)rr; q.rho = (R)rho;
  q.pp = (R)ppd;
  q.H = (R)(bEp + (double)Uq[V::E] + ppd);
  R uu = R(0);
  const R irho = inv_b(q.rho);
  for (int i = 0; i < D; ++i) {
    q.m[i] = Uq[V::M0 + i];
    q.u[i] = q.m[i] * irho;
    uu += q.u[i] * q.u[i];
  }
  const R gam = R(1) + (R)gasR * inv_b((R)Cv);
  q.cm = sqrt(gam * (R)p * irho);
  if (RAIN) {
    if (a.vr_mode == 0) q.vr = (R)a.vr_const;
    else q.vr = (R)a.vr_pref * (rr > 0.0 ? pow_b((R)rr, R(0.125)) : R(0));
    q.rrvr = q.rr * q.vr;
    q.rain_e = ((R)(a.cl * (T - a.Tref)) + R(0.5) * uu) * q.rrvr;
    q.rc = (R)rc;
    q.dvs = (R)(rvs - rv);
    q.Tm = (R)(T - a.Tref);
  } else {
    q.vr = R(0); q.rrvr = R(0); q.rain_e = R(0);
    q.rc = R(0); q.dvs = R(0); q.Tm = R(0);
  }
}

// Background at vertical index iz.
struct Bg {
  double rd, rm, p, Ep, rr, E;
};

__device__ __forceinline__ Bg bg_at(const KArgs& a, int iz) {
  const double2* b = (const double2*)a.bgt + (unsigned)iz * (kBgStride / 2);
  const double2 x = b[0], y = b[1], z = b[2];
  return Bg{x.x, x.y, y.x, y.y, z.x, z.y};
}

// Full state at a node from the stored perturbation U, the background there and
// the split result (T, rho_vs(T)): rho_v = min(rho_vs, rho_m).
template <typename R, int D, int RAIN>
__device__ __forceinline__ void eval_bg(const KArgs& a, const R* Uq, double T, double rvs, const Bg& b,
                                        Pt<R, D, RAIN>& q) {
  const double rm = b.rm + (double)Uq[Vars<D, RAIN>::RM];
  eval_core<R, D, RAIN>(a, Uq, T, fmin(rvs, rm), rvs, b.rd, b.rm, RAIN ? b.rr : 0.0, b.p, b.Ep, q);
}

template <typename R, int D, int RAIN>
__device__ __forceinline__ void eval_point(const KArgs& a, const R* Uq, double T, double rvs, int iz,
                                           Pt<R, D, RAIN>& q) {
  eval_bg<R, D, RAIN>(a, Uq, T, rvs, bg_at(a, iz), q);
}

// Physical flux in direction j (Section 2.3 perturbation form).
template <typename R, int D, int RAIN, int J>
__device__ __forceinline__ void flux(const Pt<R, D, RAIN>& q, R* F) {
  using V = Vars<D, RAIN>;
  constexpr bool VERT = (J == D - 1);
  const R uj = q.u[J];
  F[V::RD] = q.rd * uj;
  F[V::RM] = q.rm * uj;
  if (RAIN) F[V::RR] = VERT ? q.rr * uj - q.rrvr : q.rr * uj;
#pragma unroll
  for (int i = 0; i < D; ++i) {
    R f = q.m[i] * uj;
    if (i == J) f += q.pp;
    if (RAIN && VERT) f -= q.rrvr * q.u[i];
    F[V::M0 + i] = f;
  }
  F[V::E] = (RAIN && VERT) ? q.H * uj - q.rain_e : q.H * uj;
}

template <typename R, int D, int RAIN, int J>
__device__ __forceinline__ R wave_speed(const Pt<R, D, RAIN>& q) {
  R l = fabs(q.u[J]) + q.cm;
  if (RAIN && J == D - 1) l += fabs(q.vr);
  return l;
}

// Slip-wall ghost (Section 3.2): momentum reflected in the wall normal e_j.
template <typename R, int D, int RAIN, int J>
__device__ __forceinline__ void reflect(Pt<R, D, RAIN>& q) {
  q.m[J] = -q.m[J];
  q.u[J] = -q.u[J];
}

// Sources: gravity on the vertical momentum and the energy (Section 2.3),
// Kessler warm rain (Section 2.1) moving mass between rho_m and rho_r.
template <typename R, int D, int RAIN>
__device__ __forceinline__ void sources(const KArgs& a, const R* Uq, const Pt<R, D, RAIN>& q, R* G) {
  using V = Vars<D, RAIN>;
  R rhop = Uq[V::RD] + Uq[V::RM];
  if (RAIN) rhop += Uq[V::RR];
  G[V::M0 + D - 1] -= rhop * (R)a.g;
  G[V::E] -= q.rho * (R)a.g * q.u[D - 1];
  if (RAIN) {
    const R rrp = q.rr > R(0) ? q.rr : R(0);
    R p316 = R(0), p12 = R(0), p78 = R(0);
    if (rrp > R(0)) {
      kessler_pow(rrp, p316, p12, p78);
    }
    const R Sev = (R(3.86e-3) - R(9.41e-5) * q.Tm) * (R(1) + R(9.1) * p316) * q.dvs * p12;
    const R au = q.rc - (R)a.q_au * q.rho;
    const R Sau = au > R(0) ? R(1e-3) * au : R(0);
    const R Sac = R(1.72) * q.rc * p78;
    const R S = Sev - Sau - Sac;
    G[V::RM] += S;
    G[V::RR] -= S;
  }
}

}  // namespace dgm
