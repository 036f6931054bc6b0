// Adjoint kernels of libdgmoist: vector-Jacobian products of the right-hand
// side, of the implicit-condensation split and of an SSP-RK stage.
//
// The pointwise reverse pass recomputes the forward quantities of one node in
// FP64 and propagates adjoints back through the fluxes, the wave speed, the
// sources, the equation of state and the split.  The split's derivative is
// the implicit-function derivative of the root (Section 2.2 system):
//   saturated:   f(T; rd, rm, rr, re) = 0  =>  dT = -(df/dtheta) dtheta / f_T,
//                rho_v = rho_vs(T);
//   unsaturated: T = T_ref + (re - rm (L - R_v T_ref)) / (c_vd rd + c_vv rm + c_l rr),
//                rho_v = rm.
// At kinks the active branch is differentiated: ties of the split go to the
// unsaturated branch, ties of the face maximum to the minus side, sign(0) = 0,
// and clamps at zero have derivative 0 there.
#pragma once
#include "dg_kernels.h"

namespace dgm {

// Reverse pass of the split: adjoints (Tb, rvb) of (T, rho_v) -> adjoints of
// (rd, rm, rr, re), added to the outputs.  `sat` is the branch of the forward
// split; T and rvs = rho_vs(T) come from it.
__device__ __forceinline__ void split_reverse(const KArgs& a, bool sat, double rd, double rm, double rr,
                                              double T, double rvs, double Tb, double rvb,
                                              double& rdb, double& rmb, double& rrb, double& reb) {
  const double Tm = T - a.Tref;
  if (!sat) {
    const double Cu = a.cvd * rd + a.cvv * rm + a.cl * rr;
    const double t = Tb * rcp64(Cu);
    reb += t;
    rmb += t * (-a.Lp - a.cvv * Tm) + rvb;
    rdb += -t * a.cvd * Tm;
    rrb += -t * a.cl * Tm;
    return;
  }
  const double dc = a.cvv - a.cl;
  const double Cv = a.cvd * rd + a.cvv * rvs + a.cl * (rm - rvs + rr);
  const double iT = rcp64(T);
  const double drvs = rvs * (a.am1 + a.b * iT) * iT;
  const double fT = Cv + drvs * (dc * Tm + a.Lp);
  const double tt = (Tb + rvb * drvs) * rcp64(fT);
  reb += tt;
  rdb += -tt * a.cvd * Tm;
  rmb += -tt * a.cl * Tm;
  rrb += -tt * a.cl * Tm;
}

// Reverse pass of one node.  The forward quantities are recomputed in FP64 and
// the fluxes' adjoints are folded direction by direction into the node's
// accumulators, so the seeds of one direction only are live (held for all
// three at once, with the wall ghosts' own reverse passes, the kernel took
// 375 registers: one wavefront per SIMD).  Bound by FP64 issue and latency at
// two wavefronts per SIMD (193 registers): a tendency and its product on 40 x 36 x
// 20 Q3 (FP32) 358 -> 204 us.
template <int D, int RAIN>
struct Reverse {
  using V = Vars<D, RAIN>;
  static constexpr int NV = V::NV, Z = D - 1;
  // forward
  double rd, rm, rr, rho, irho, m[D], u[D], uu, E, T, Tm, rvs, rv, rc, Rg, p, pp, iCv, gam, H, c2, cm, vr, X;
  bool sat;
  // adjoints
  double rdb, rmb, rrb, rhob, Eb, Tb, rvb, ppb, Hb, cmb, vrb, mb[D], ub[D];

  template <typename R>
  __device__ __forceinline__ void forward(const KArgs& a, const R* Uq, double T_, double rvs_, const Bg& bg) {
    T = T_;
    rvs = rvs_;
    rd = bg.rd + (double)Uq[V::RD];
    rm = bg.rm + (double)Uq[V::RM];
    rr = RAIN ? bg.rr + (double)Uq[V::RR] : 0.0;
    rho = rd + rm + rr;
    irho = rcp64(rho);
    uu = 0.0;
#pragma unroll
    for (int i = 0; i < D; ++i) {
      m[i] = (double)Uq[V::M0 + i];
      u[i] = m[i] * irho;
      uu += u[i] * u[i];
    }
    E = bg.E + (double)Uq[V::E];
    sat = rvs < rm;
    rv = sat ? rvs : rm;
    rc = rm - rv;
    Rg = rd * a.Rd + rv * a.Rv;
    p = Rg * T;
    pp = p - bg.p;
    const double Cv = a.cvd * rd + a.cvv * rv + a.cl * (rc + rr);
    iCv = rcp64(Cv);
    gam = 1.0 + Rg * iCv;
    c2 = gam * p * irho;
    cm = sqrt(c2);
    H = E + p;
    Tm = T - a.Tref;
    vr = 0.0;
    if (RAIN) vr = (a.vr_mode == 0) ? a.vr_const : (rr > 0.0 ? a.vr_pref * pow(rr, 0.125) : 0.0);
    X = a.cl * Tm + 0.5 * uu;            // rain energy factor
    rdb = rmb = rrb = rhob = Eb = Tb = rvb = ppb = Hb = cmb = vrb = 0.0;
#pragma unroll
    for (int i = 0; i < D; ++i) mb[i] = ub[i] = 0.0;
  }

  // direction J: adjoints Fb of the flux without the rain's fall, Wb of the
  // fall's part (vertical direction only) and lb of the wave speed
  template <int J>
  __device__ __forceinline__ void flux_reverse(const KArgs& a, const double* Fb, const double* Wb, double lb) {
    constexpr bool vert = (J == Z);
    rdb += Fb[V::RD] * u[J];
    rmb += Fb[V::RM] * u[J];
    if (RAIN) rrb += Fb[V::RR] * u[J];
    double uJ = Fb[V::RD] * rd + Fb[V::RM] * rm + Fb[V::E] * H;
    if (RAIN) uJ += Fb[V::RR] * rr;
#pragma unroll
    for (int i = 0; i < D; ++i) {
      mb[i] += Fb[V::M0 + i] * u[J];
      uJ += Fb[V::M0 + i] * m[i];
    }
    ppb += Fb[V::M0 + J];
    Hb += Fb[V::E] * u[J];
    // wave speed |u_J| + v_r [J vertical] + c_m
    uJ += lb * (u[J] > 0.0 ? 1.0 : (u[J] < 0.0 ? -1.0 : 0.0));
    cmb += lb;
    ub[J] += uJ;
    if (RAIN && vert) {
      // fall: -rho_r v_r (1, u, X) on rho_r, m, E
      double s = Wb[V::RR] + Wb[V::E] * X;
      const double f = rr * vr;
#pragma unroll
      for (int i = 0; i < D; ++i) {
        s += Wb[V::M0 + i] * u[i];
        ub[i] -= (Wb[V::M0 + i] + Wb[V::E] * u[i]) * f;
      }
      rrb -= s * vr;
      vrb += lb - s * rr;
      Tb -= Wb[V::E] * a.cl * f;
    }
  }

  // sources (adjoints Gb), equation of state, split; adds to Ub
  __device__ __forceinline__ void finish(const KArgs& a, const double* Gb, double* Ub) {
    // gravity
    {
      const double gz = Gb[V::M0 + Z] * a.g;
      rdb -= gz;   // rho' = rho_d' + rho_m' + rho_r'
      rmb -= gz;
      if (RAIN) rrb -= gz;
      const double ge = Gb[V::E] * a.g;
      rhob -= ge * u[Z];
      ub[Z] -= ge * rho;
    }
    // Kessler
    if (RAIN) {
      const double Sb = Gb[V::RM] - Gb[V::RR];
      const double dvs = rvs - rv;                    // 0 on the saturated branch
      double rcb = 0.0, dvsb = 0.0, ip12 = 0.0;
      if (rr > 0.0) {
        const double Aev = 3.86e-3 - 9.41e-5 * Tm;
        double p316, p12, p78;
        kessler_pow(rr, p316, p12, p78);
        // (1/rr only by halves: it overflows for the thinnest rain, its square root does not)
        ip12 = rcp64(p12);
        const double Bev = 1.0 + 9.1 * p316;
        Tb += Sb * (-9.41e-5) * Bev * dvs * p12;
        dvsb += Sb * Aev * Bev * p12;
        // p12' = p12 / (2 rr), p316' = 3/16 p316 / rr, p78' = 7/8 p78 / rr
        rrb += Sb * (Aev * dvs * ip12 * (9.1 * 0.1875 * p316 + 0.5 * Bev) - 1.72 * 0.875 * rc * (p78 * ip12 * ip12));
        rcb -= Sb * 1.72 * p78;
      }
      if (rc - a.q_au * rho > 0.0) {                    // autoconversion
        rcb -= Sb * 1e-3;
        rhob += Sb * 1e-3 * a.q_au;
      }
      if (!sat) {                                       // dvs = rho_vs(T) - rm
        const double iT = rcp64(T);
        Tb += dvsb * rvs * (a.am1 + a.b * iT) * iT;
        rmb -= dvsb;
      }
      rmb += rcb;
      rvb -= rcb;
      if (a.vr_mode != 0 && rr > 0.0) rrb += vrb * (vr * 0.125 * ip12 * ip12);
    }
    // H = E + p, p' = p - p_bar
    Eb += Hb;
    double pb = Hb + ppb;
    // c_m = sqrt(gamma p / rho), gamma = 1 + Rg / Cv
    {
      const double c2b = cmb * 0.5 * rcp64(cm);
      const double gb = c2b * p * irho;
      pb += c2b * gam * irho;
      rhob -= c2b * c2 * irho;
      const double Rgb = gb * iCv;
      const double Cvb = -Rgb * Rg * iCv;
      rdb += Rgb * a.Rd + Cvb * a.cvd;
      rvb += Rgb * a.Rv + Cvb * (a.cvv - a.cl);
      rmb += Cvb * a.cl;
      rrb += Cvb * a.cl;
    }
    // p = (rd R_d + rv R_v) T
    rdb += pb * a.Rd * T;
    rvb += pb * a.Rv * T;
    Tb += pb * Rg;
    // u_i = m_i / rho
#pragma unroll
    for (int i = 0; i < D; ++i) {
      const double t = ub[i] * irho;
      mb[i] += t;
      rhob -= t * u[i];
    }
    // split: (rd, rm, rr, re) -> (T, rv)
    double reb = 0.0;
    split_reverse(a, sat, rd, rm, rr, T, rvs, Tb, rvb, rdb, rmb, rrb, reb);
    // re = E - |m|^2 / (2 rho)
    Eb += reb;
#pragma unroll
    for (int i = 0; i < D; ++i) mb[i] -= reb * u[i];
    rhob += reb * 0.5 * uu;
    // rho = rd + rm + rr
    Ub[V::RD] += rdb + rhob;
    Ub[V::RM] += rmb + rhob;
    if (RAIN) Ub[V::RR] += rrb + rhob;
#pragma unroll
    for (int i = 0; i < D; ++i) Ub[V::M0 + i] += mb[i];
    Ub[V::E] += Eb;
  }
};

// ---------------------------------------------------------------------------
// adjoint of the right-hand side
// ---------------------------------------------------------------------------
// What a node reads for its face in direction J: the neighbour's matching node
// (on a wall, and for a node off the J-faces, the own one; then unused).
template <typename R, int D, int RAIN>
struct FaceVjp {
  R U[Vars<D, RAIN>::NV], L[Vars<D, RAIN>::NV];
  double T, rvs;
  int izn;
  bool face, wall;
};

template <typename R, int K, int D, int RAIN, int J>
__device__ __forceinline__ void face_load(const Item& item, const ElemCoord<D>& ec, int ij, int iz, bool active,
                                          unsigned g, unsigned N, const R* __restrict__ U, const double* __restrict__ auxT,
                                          const double* __restrict__ auxS, const R* __restrict__ lam,
                                          FaceVjp<R, D, RAIN>& f) {
  using S = Shape<K, D, block_threads<R>()>;
  constexpr int P1 = S::P1, NP = S::NP, NV = Vars<D, RAIN>::NV;
  constexpr int STR = (J == 0) ? 1 : (J == 1 ? P1 : P1 * P1);
  const bool plus = ij == K;
  const int c = ec.c[J], n = item.n[J];
  const bool at_end = plus ? c == n - 1 : c == 0;
  // (a thread past the item's end holds no face node: in FP32 it reads the item's
  // first node throughout, in FP64 the buffer's bounds check covers what it reads)
  f.face = (sizeof(R) == 8 || active) && (ij == 0 || ij == K);
  f.wall = f.face && at_end && item.bc[J] == 1;
  const int step = at_end ? (plus ? 1 - n : n - 1) : (plus ? 1 : -1);
  const bool nb = f.face && !f.wall;
  const unsigned gn = nb ? g + (unsigned)(step * elem_stride(item, J) * NP + (plus ? -K * STR : K * STR)) : g;
#pragma unroll
  for (int v = 0; v < NV; ++v) f.U[v] = ld(U, N, v, gn);
#pragma unroll
  for (int v = 0; v < NV; ++v) f.L[v] = ld(lam, N, v, gn);
  f.T = ld_f64<R>(auxT, N, gn);
  f.rvs = ld_f64<R>(auxS, N, gn);
  f.izn = J == D - 1 && nb ? item.hoff + (c + step) * P1 + (plus ? 0 : K) : iz;
}

// One direction: the volume term's transposed contraction, the node's face in
// it (the adjoint of the Lax-Friedrichs flux, its jump term straight into Ub),
// and the reverse pass of the flux.  sL: the adjoint of dU/dt in the block's
// LDS tile (FP64), sD the weak-form matrix.
//
// On a slip wall the flux is (F(U) + F(g U))/2 + Lambda (U - g U)/2 with g the
// mirror; the two fluxes differ in sign except for the normal momentum (equal)
// and the rain's fall (equal), so the ghost needs no reverse pass of its own.
template <typename R, int K, int D, int RAIN, int J>
__device__ __forceinline__ void direction_vjp(const KArgs& a, const MemberDesc& md, int t, int ij, const double* sL,
                                              const double* sD, const R* Uq, const R* Lq, R lo,
                                              const FaceVjp<R, D, RAIN>& f, Reverse<D, RAIN>& rev, double* Ub) {
  using S = Shape<K, D, block_threads<R>()>;
  using V = Vars<D, RAIN>;
  constexpr int P1 = S::P1, NV = V::NV, NT = S::NT;
  constexpr int STR = (J == 0) ? 1 : (J == 1 ? P1 : P1 * P1);
  double Fb[NV], Wb[NV], lb = 0.0;
  {
    const int base = t - ij * STR;
    const double s = md.two_over_h[J];
    double d[P1];
#pragma unroll
    for (int b = 0; b < P1; ++b) d[b] = s * sD[b * P1 + ij];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double acc = 0.0;
#pragma unroll
      for (int b = 0; b < P1; ++b) acc += d[b] * sL[v * NT + base + b * STR];
      Fb[v] = Wb[v] = acc;
    }
  }
  if (f.face) {
    const bool plus = ij == K;     // own node on its +J face: own side is K-
    const double lift = md.lift[J][0];   // (the Lobatto weights are symmetric)
    const double sgn = plus ? 0.5 : -0.5;
    R qnU[NV];
    R ln = lo;
    if (!f.wall) {
#pragma unroll
      for (int v = 0; v < NV; ++v) qnU[v] = f.U[v];
      Pt<R, D, RAIN> qn;
      eval_point<R, D, RAIN>(a, qnU, f.T, f.rvs, f.izn, qn);
      ln = wave_speed<R, D, RAIN, J>(qn);
    }
    // F* = (F(U-) + F(U+)).n / 2 + Lambda (U- - U+) / 2, Lambda = max(l-, l+),
    // ties to the minus side
    const bool own = f.wall || (plus ? lo >= ln : lo > ln);
    const double Lam = own ? (double)lo : (double)ln;
    double jump = 0.0;           // Fsb . (own - neighbour)
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const bool nrm = v == V::M0 + J;
      // adjoint of F*: R(K-) -= lift F*, R(K+) += lift F*
      const double Fsb = (plus ? -lift : lift) * ((double)Lq[v] - (f.wall ? 0.0 : (double)f.L[v]));
      const double Un = f.wall ? (nrm ? -(double)Uq[v] : (double)Uq[v]) : (double)f.U[v];
      jump += Fsb * ((double)Uq[v] - Un);
      Fb[v] += f.wall ? (nrm ? Fsb : 0.0) : 0.5 * Fsb;
      Wb[v] += f.wall ? (nrm ? 0.0 : Fsb) : 0.5 * Fsb;
      Ub[v] += (f.wall ? (nrm ? 2.0 : 0.0) : 1.0) * sgn * Lam * Fsb;
    }
    if (own) lb = sgn * jump;
  }
  rev.template flux_reverse<J>(a, Fb, Wb, lb);
}

// Wavefronts per SIMD that the registers are bound to: two, but one at 3D Q1 with
// rain in FP64, where two spill 78 registers (64 x 60 x 30 164 -> 128 us; in FP32,
// which spills 35, 114 and 112).  The other shapes measured the same or slower at one.
template <typename R, int K, int D, int RAIN>
constexpr int vjp_min_waves() { return sizeof(R) == 8 && K == 1 && D == 3 && RAIN ? 1 : 2; }

template <typename R, int K, int D, int RAIN>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(vjp_min_waves<R, K, D, RAIN>())))
rhs_vjp_kernel(KArgs a, const R* __restrict__ U, const double* __restrict__ auxT,
               const double* __restrict__ auxS, const R* __restrict__ lam, R* __restrict__ out,
               const R* __restrict__ X1, const R* __restrict__ X2, const double* __restrict__ dt_m,
               double cx1, double cx2, double c1, double c2) {
  using S = Shape<K, D, block_threads<R>()>;
  using V = Vars<D, RAIN>;
  constexpr int P1 = S::P1, NP = S::NP, NV = V::NV;
  __shared__ double sL[NV * S::NT];
  __shared__ double sD[P1 * P1];
  const int t = threadIdx.x;
  if (t < P1 * P1) sD[t] = (double)(R)a.Dhat[t];
  // one work item per block (no item loop: loop-invariant values would stay
  // live across the body)
  const int it_ = ItemWalk(a.nitems).item(0);
  if (it_ < 0) return;
  const Item item = a.items[it_];
  const MemberDesc& md = a.mem[item.member];
  const int le = t / NP, n = t - le * NP;
  const bool active = item.e0 + le < item.ne;
  const unsigned N = a.nnodes;
  const unsigned g = (unsigned)(item.eoff + item.e0) * NP + (active ? t : 0);
  const ElemCoord<D> ec = item_coord<D>(item, active ? le : 0);
  int idx[3];
  idx[0] = n % P1;
  idx[1] = (n / P1) % P1;
  idx[2] = (D == 3) ? n / (P1 * P1) : 0;
  const int iz = item.hoff + ec.c[D - 1] * P1 + idx[D - 1];
  R Uq[NV], Lq[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) Uq[v] = ld(U, N, v, g);
#pragma unroll
  for (int v = 0; v < NV; ++v) Lq[v] = ld(lam, N, v, g);
  const double T = ld_f64<R>(auxT, N, g), rvs = ld_f64<R>(auxS, N, g);
  const Bg bg = bg_at(a, iz);
  // a direction's neighbour values are in flight while the previous one is
  // worked on
  FaceVjp<R, D, RAIN> f;
  face_load<R, K, D, RAIN, 0>(item, ec, idx[0], iz, active, g, N, U, auxT, auxS, lam, f);
#pragma unroll
  for (int v = 0; v < NV; ++v) sL[v * S::NT + t] = (double)Lq[v];
  __syncthreads();
  if (!active) return;
  Pt<R, D, RAIN> q;
  eval_bg<R, D, RAIN>(a, Uq, T, rvs, bg, q);
  Reverse<D, RAIN> rev;
  rev.forward(a, Uq, T, rvs, bg);
  double Ub[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) Ub[v] = 0.0;
  {
    FaceVjp<R, D, RAIN> f1;
    face_load<R, K, D, RAIN, 1>(item, ec, idx[1], iz, active, g, N, U, auxT, auxS, lam, f1);
    direction_vjp<R, K, D, RAIN, 0>(a, md, t, idx[0], sL, sD, Uq, Lq, wave_speed<R, D, RAIN, 0>(q), f, rev, Ub);
    if constexpr (D == 3)
      face_load<R, K, D, RAIN, 2>(item, ec, idx[2], iz, active, g, N, U, auxT, auxS, lam, f);
    direction_vjp<R, K, D, RAIN, 1>(a, md, t, idx[1], sL, sD, Uq, Lq, wave_speed<R, D, RAIN, 1>(q), f1, rev, Ub);
  }
  if constexpr (D == 3)
    direction_vjp<R, K, D, RAIN, 2>(a, md, t, idx[2], sL, sD, Uq, Lq, wave_speed<R, D, RAIN, 2>(q), f, rev, Ub);
  // sources: dU/dt = ... + G
  double Gb[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) Gb[v] = (double)Lq[v];
  rev.finish(a, Gb, Ub);
  // out = cx1 X1 + cx2 X2 + c1 lam + c2 dt (d rhs/dU)^T lam
  const double k2 = c2 * (dt_m ? dt_m[item.member] : 1.0);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    double o = c1 * (double)Lq[v] + k2 * Ub[v];
    if (X1) o += cx1 * (double)ld(X1, N, v, g);
    if (X2) o += cx2 * (double)ld(X2, N, v, g);
    st(out, N, v, g, (R)o);
  }
}

// adjoint of the split alone: (T_bar, rho_v_bar, rho_c_bar) -> U_bar
template <typename R, int K, int D, int RAIN>
__global__ void __launch_bounds__(256)
split_vjp_kernel(KArgs a, const R* __restrict__ U, const double* __restrict__ auxT,
                 const double* __restrict__ auxS, const double* __restrict__ Tbar,
                 const double* __restrict__ rvbar, const double* __restrict__ rcbar,
                 R* __restrict__ out) {
  using S = Shape<K, D, block_threads<R>()>;
  using V = Vars<D, RAIN>;
  constexpr int P1 = S::P1, NP = S::NP, NV = V::NV;
  const ItemWalk walk(a.nitems);
  for (int kk = 0;; ++kk) {
  const int it_ = walk.item(kk);
  if (it_ < 0) break;
  const int t = threadIdx.x;
  const Item item = a.items[it_];
  const MemberDesc& md = a.mem[item.member];
  const int le = t / NP, n = t - le * NP;
  const int e = item.e0 + le;
  if (e >= item.ne) continue;
  const unsigned N = a.nnodes;
  const unsigned g = (unsigned)(item.eoff + e) * NP + n;
  const ElemCoord<D> ec = item_coord<D>(item, le);
  const int l = (D == 2) ? n / P1 : n / (P1 * P1);
  const int iz = item.hoff + ec.c[D - 1] * P1 + l;
  double Uq[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) Uq[v] = (double)(U + (size_t)v * N)[g];
  const Bg bg = bg_at(a, iz);
  const double rd = bg.rd + Uq[V::RD];
  const double rm = bg.rm + Uq[V::RM];
  const double rr = RAIN ? bg.rr + Uq[V::RR] : 0.0;
  const double irho = rcp64(rd + rm + rr);
  double uu = 0.0, u[D];
#pragma unroll
  for (int i = 0; i < D; ++i) {
    u[i] = Uq[V::M0 + i] * irho;
    uu += u[i] * u[i];
  }
  const double T = auxT[g], rvs = auxS[g];
  const bool sat = rvs < rm;
  const double Tb = Tbar ? Tbar[g] : 0.0;
  const double rcb = rcbar ? rcbar[g] : 0.0;
  const double rvb = (rvbar ? rvbar[g] : 0.0) - rcb;   // rho_c = rm - rho_v
  double rdb = 0, rmb = rcb, rrb = 0, reb = 0;
  split_reverse(a, sat, rd, rm, rr, T, rvs, Tb, rvb, rdb, rmb, rrb, reb);
  double Ub[NV];
  double rhob = reb * 0.5 * uu;
  Ub[V::RD] = rdb + rhob;
  Ub[V::RM] = rmb + rhob;
  if (RAIN) Ub[V::RR] = rrb + rhob;
#pragma unroll
  for (int i = 0; i < D; ++i) Ub[V::M0 + i] = -reb * u[i];
  Ub[V::E] = reb;
#pragma unroll
  for (int v = 0; v < NV; ++v) (out + (size_t)v * N)[g] = (R)Ub[v];
  }
}

}  // namespace dgm
