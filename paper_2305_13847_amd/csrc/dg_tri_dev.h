// Device code on triangulations: the space P^k of Section 3.1 on a conforming
// triangulation of the vertical plane.
//
// A block holds a few elements with one thread per volume point of each
// (Duffy-mapped rule of the footnote in Section 3.4); coefficients and
// per-point results are exchanged through LDS, and a face point's thread
// gathers the neighbour's coefficients through the neighbour table to form
// the neighbour's trace at the shared point (Section 3.2).  The reference
// tables sit in constant memory.
//
// Precision as on the box meshes: the state, fluxes and accumulation in R,
// the reconstruction of full densities and p', the split and the projected T
// and rho_v in FP64.
#pragma once
#include <type_traits>

#include "dg_device.h"

namespace dgm {

template <int K>
struct TriShape {
  static constexpr int NP = (K + 1) * (K + 2) / 2;   // modes
  static constexpr int NQ = (K + 1) * (K + 2);       // volume points
  static constexpr int NF = K + 1;                   // points per face
  // rows of NP values padded to whole 16-byte LDS reads (single and double)
  static constexpr int NPP = (NP + 3) / 4 * 4, NPD = (NP + 1) / 2 * 2;
};

// Reference tables of order K (filled on the host at handle creation).
template <typename R, int K>
struct alignas(16) TriTab {
  static constexpr int NP = TriShape<K>::NP, NQ = TriShape<K>::NQ, NF = TriShape<K>::NF;
  static constexpr int NPP = TriShape<K>::NPP, NPD = TriShape<K>::NPD;
  R psi[NQ][NPP];                           // basis at the volume points
  R g3[NQ][NP][4];                          // its reference gradient (r, s) and value, together
  double psid[NQ][NPD];                     // the basis in FP64 (T, rho_v, split, projection)
  R psif[3][NF][NPP];                       // basis at the face points
  double psifd[3][NF][NPD];
  double wd[NQ];                            // volume weights (sum 1/2)
  double rq[NQ], sq[NQ];                    // volume points
  double rf[3][NF], sf[3][NF];              // face points
  R w[(NQ + 3) / 4 * 4];                    // volume weights
  R wf[(NF + 3) / 4 * 4];                   // half the face Gauss weights
};

__constant__ TriTab<float, 1> c_tri_f1;
__constant__ TriTab<float, 2> c_tri_f2;
__constant__ TriTab<float, 3> c_tri_f3;
__constant__ TriTab<float, 4> c_tri_f4;
__constant__ TriTab<double, 1> c_tri_d1;
__constant__ TriTab<double, 2> c_tri_d2;
__constant__ TriTab<double, 3> c_tri_d3;
__constant__ TriTab<double, 4> c_tri_d4;

template <typename R, int K>
__device__ __forceinline__ const TriTab<R, K>& ttab() {
  if constexpr (sizeof(R) == 4) {
    if constexpr (K == 1) return c_tri_f1;
    else if constexpr (K == 2) return c_tri_f2;
    else if constexpr (K == 3) return c_tri_f3;
    else return c_tri_f4;
  } else {
    if constexpr (K == 1) return c_tri_d1;
    else if constexpr (K == 2) return c_tri_d2;
    else if constexpr (K == 3) return c_tri_d3;
    else return c_tri_d4;
  }
}

struct TriArgs {
  const double* xy;   // ne x 3 x (x, z)
  const int* nbr;     // ne x 3: neighbour * 4 + its face; -1 slip wall
  const int* layer;   // ne: the background layer that holds the centroid
  // background: per layer the degree-K interpolant through its Gauss heights as
  // coefficients of xi^i on [-1, 1], fields (rho_d, rho_m, p, E + p, rho_r, E)
  const double* bgm;
  double z0, inv_dz;
  int ne;
};

// Vertex heights and layer of element e.
struct TriZ {
  double z0, dz1, dz2;
  int layer;
};

__device__ __forceinline__ TriZ tri_z(const TriArgs& t, int e) {
  const double* v = t.xy + (size_t)e * 6;
  TriZ g;
  g.z0 = v[1];
  g.dz1 = v[3] - v[1];
  g.dz2 = v[5] - v[1];
  g.layer = t.layer[e];
  return g;
}

// Background at height z from layer l's interpolant.
template <int K>
__device__ __forceinline__ Bg tri_bg(const TriArgs& t, int l, double z) {
  const double xi = 2.0 * ((z - t.z0) * t.inv_dz - (double)l) - 1.0;
  const double2* c = (const double2*)t.bgm + (size_t)l * (3 * (K + 1));
  double2 x = c[3 * K], y = c[3 * K + 1], w = c[3 * K + 2];
#pragma unroll
  for (int i = K - 1; i >= 0; --i) {
    const double2 a = c[3 * i], b = c[3 * i + 1], d = c[3 * i + 2];
    x.x = fma(x.x, xi, a.x); x.y = fma(x.y, xi, a.y);
    y.x = fma(y.x, xi, b.x); y.y = fma(y.y, xi, b.y);
    w.x = fma(w.x, xi, d.x); w.y = fma(w.y, xi, d.y);
  }
  return Bg{x.x, x.y, y.x, y.y, w.x, w.y};
}

// The flux of Section 2.3 along the direction (nx, nz): F(q) . n for every
// variable (n need not be a unit vector).
template <typename R, int RAIN>
__device__ __forceinline__ void flux_dir(const Pt<R, 2, RAIN>& q, R nx, R nz, R* Fn) {
  using V = Vars<2, RAIN>;
  const R un = q.u[0] * nx + q.u[1] * nz;
  Fn[V::RD] = q.rd * un;
  Fn[V::RM] = q.rm * un;
  R f0 = q.m[0] * un + q.pp * nx, f1 = q.m[1] * un + q.pp * nz, fe = q.H * un;
  if (RAIN) {
    const R fall = q.rrvr * nz;
    Fn[V::RR] = q.rr * un - fall;
    f0 -= fall * q.u[0];
    f1 -= fall * q.u[1];
    fe -= q.rain_e * nz;
  }
  Fn[V::M0] = f0;
  Fn[V::M0 + 1] = f1;
  Fn[V::E] = fe;
}

// wave speed along the unit normal (Section 3.2): |u.n| + |v_r n_z| + c_m
template <typename R, int RAIN>
__device__ __forceinline__ R speed_dir(const Pt<R, 2, RAIN>& q, R nx, R nz) {
  R l = fabs(q.u[0] * nx + q.u[1] * nz) + q.cm;
  if (RAIN) l += fabs(q.vr * nz);
  return l;
}

// Split (Section 2.2) of the state with perturbation Uq (FP64) over background
// b at one point, from the guess Tg: T and rho_v = min(rho_vs(T), rho_m).
template <int RAIN>
__device__ __forceinline__ SplitOut tri_split_point(const KArgs& a, const double* Uq, const Bg& b, double Tg,
                                                    double* rv) {
  using V = Vars<2, RAIN>;
  const double rd = b.rd + Uq[V::RD];
  const double rm = b.rm + Uq[V::RM];
  const double rr = RAIN ? b.rr + Uq[V::RR] : 0.0;
  const double m0 = Uq[V::M0], m1 = Uq[V::M0 + 1];
  const double re = (b.E + Uq[V::E]) - 0.5 * (m0 * m0 + m1 * m1) * rcp64(rd + rm + rr);
  const SplitOut s = split_scratch(a, rd, rm, rr, re, Tg);
  *rv = fmin(s.rvs, rm);
  return s;
}

// eval_core with the background of tri_bg
template <typename R, int RAIN>
__device__ __forceinline__ void tri_eval(const KArgs& a, const R* U, double T, double rv, const Bg& b,
                                         Pt<R, 2, RAIN>& q) {
  eval_core<R, 2, RAIN>(a, U, T, rv, RAIN ? rho_vs(a, T) : 0.0, b.rd, b.rm, RAIN ? b.rr : 0.0, b.p, b.Ep, q);
}

// Work layout: a block of 256 threads holds EPB elements, one thread per
// volume point of each (EPB NQ threads; the rest idle).  The elements'
// coefficients, their projected T and rho_v and the per-point results sit in
// LDS, in rows padded to 16-byte reads; the contractions between modes and
// points read them from there:
//   points:  thread (element, q) evaluates the state at volume point q, its
//            flux along the two columns of A^{-T} and its sources;
//   modes:   thread (element, m + half NP) sums all variables of mode m over
//            half of the volume points; the halves then exchange partial sums
//            and each finishes half of the variables (faces, update);
//   faces:   thread (element, j), j < 3 NF, handles face point j: its own
//            trace from LDS, the neighbour's from coefficients parked there.
// Bound by instruction issue and LDS latency.  At 256 x 128 x 2, P3, FP32 a
// stage took 133 us with 2503 VALU instructions per wavefront, a third of them
// index arithmetic (one division chain per loaded value), Lagrange weights of
// the background evaluated twice per point, conversions in the split, and
// single-word LDS reads; now 88 us with 1460.  The LDS is busy nearly as long as
// the VALU: rows of several elements in the same banks alone cost 4 of 92 us.
template <int K>
struct TriBlock {
  static constexpr int NQ = TriShape<K>::NQ;
  static constexpr int EPB = 256 / NQ;
  static constexpr int NT = EPB * NQ;
};

template <typename R, int K, int RAIN>
struct TriLds {
  static constexpr int NV = Vars<2, RAIN>::NV, NP = TriShape<K>::NP, NQ = TriShape<K>::NQ;
  static constexpr int NPP = TriShape<K>::NPP, NPD = TriShape<K>::NPD;
  static constexpr int NF = TriShape<K>::NF, EPB = TriBlock<K>::EPB;
  static constexpr int NVP = (NV + 3) / 4 * 4, PF = (3 * NV + 3) / 4 * 4;
  // Values after an element's rows that shift the next one's banks: a wavefront
  // reads the same row of several elements at once, and NQ PF is a multiple of 64
  // words at P2 and P3.  Without the shift, steps in FP64 take 1 to 9 % more (P2 910
  // -> 995 us on 300 x 150 x 2, P1 719 -> 770) and in FP32 at P2 and P3 4 to 5 %;
  // rain and P4 do not care.  At P1 in FP32 it costs a fourth block per CU on large
  // meshes (400 x 200 x 2, two steps: 473 us with it, 453 without) and pays on small
  // ones (8 x 4 x 2, five steps: 179 and 185.5 us).
  static constexpr int SHIFT = 4;
  // the reference tables (FP32; in FP64 they would halve the blocks per CU and
  // stay in constant memory)
  struct Empty {};
  std::conditional_t<sizeof(R) == 4, TriTab<R, K>, Empty> tab;
  alignas(16) double aux[EPB][2][NPD];   // projected T and rho_v of the stage input
  alignas(16) double ts[EPB][NQ][2];     // the weighted split of the updated state at the volume points
  alignas(16) R c[EPB][NV][NPP];         // coefficients of the stage input
  union {
    // per volume point: w F.G0, w F.G1, w G, and the shift
    alignas(16) R pf[EPB][NQ * PF + SHIFT];
    struct {                             // then the neighbours across the three faces
      alignas(16) double aux[EPB][3][2][NPD];
      alignas(16) R c[EPB][3][NV][NPP];
    } nb;
    alignas(16) double cd[EPB][NV][NPD]; // then the updated coefficients, for the split
  } u;
  union {
    alignas(16) R px[EPB][NP][NVP];      // partial sums of the modes
    alignas(16) R ff[EPB][3 * NF * NVP + SHIFT];  // then per face point the weighted normal flux
  } f;
  TriZ fz[EPB];             // heights of the vertices and background layer
  R fn[EPB][3][3];          // per face: n_x, n_z, |e_f| / det A
};

// First element of this block.  Consecutive blocks go round-robin to the 8
// XCDs; XCD x takes the contiguous block range [x per, (x+1) per), so an
// element and its neighbours in the rows above and below share an L2.  The
// grid is 8 per blocks; a block past the end returns -1 (uniformly).
template <int K>
__device__ __forceinline__ long long tri_first_element(int ne) {
  constexpr int EPB = TriBlock<K>::EPB;
  const int nblocks = (ne + EPB - 1) / EPB;
  const int per = (nblocks + 7) >> 3;
  const int b = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  return b < nblocks ? (long long)b * EPB : -1;
}

// LDS of the split kernel: coefficients and the split values only
template <typename R, int K, int RAIN>
struct TriLdsSplit {
  static constexpr int NV = Vars<2, RAIN>::NV, NQ = TriShape<K>::NQ, NPD = TriShape<K>::NPD;
  static constexpr int EPB = TriBlock<K>::EPB;
  struct Empty {};
  std::conditional_t<sizeof(R) == 4, TriTab<R, K>, Empty> tab;
  alignas(16) double ts[EPB][NQ][2];
  struct {
    alignas(16) double cd[EPB][NV][NPD];
  } u;
};

// Copy the reference tables (a plain struct) from constant memory into LDS
// (FP32 kernels), and the tables a kernel reads: the LDS copy or constant memory.
template <typename R, int K, typename L>
__device__ __forceinline__ void tri_copy_tab(L& S) {
  if constexpr (sizeof(R) == 4) {
    static_assert(sizeof(TriTab<R, K>) % 4 == 0, "tables are whole words");
    const unsigned* s = reinterpret_cast<const unsigned*>(&ttab<R, K>());
    unsigned* d = reinterpret_cast<unsigned*>(&S.tab);
    for (int i = threadIdx.x; i < (int)(sizeof(TriTab<R, K>) / 4); i += blockDim.x) d[i] = s[i];
  }
}

template <typename R, int K, typename L>
__device__ __forceinline__ const TriTab<R, K>& tri_tab(const L& S) {
  if constexpr (sizeof(R) == 4) return S.tab;
  else return ttab<R, K>();
}

// The split of the state S.u.cd at volume point q of element slot el (thread
// (el, q)), from the guess Tg, weighted, to S.ts.
template <typename R, int K, int RAIN, typename L>
__device__ __forceinline__ void tri_split_at(const KArgs& a, L& S, int el, int q, const Bg& b, double Tg, int* iters,
                                             int* bad) {
  constexpr int NV = Vars<2, RAIN>::NV, NP = TriShape<K>::NP;
  const auto& T = tri_tab<R, K>(S);
  double X[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    double s = 0.0;
#pragma unroll
    for (int m = 0; m < NP; ++m) s += S.u.cd[el][v][m] * T.psid[q][m];
    X[v] = s;
  }
  double rv;
  const SplitOut o = tri_split_point<RAIN>(a, X, b, Tg, &rv);
  S.ts[el][q][0] = o.T * T.wd[q];
  S.ts[el][q][1] = rv * T.wd[q];
  *iters = o.iters;
  *bad = o.bad;
}

// The L2 projections of the split values onto P^k, by thread (el, m + c NP)
// (c = 0: T, 1: rho_v), stored to Tn / Rn.
template <typename R, int K, int RAIN, typename L>
__device__ __forceinline__ void tri_project_split(const L& S, int el, int m, int c, long long e, bool act,
                                                  double* __restrict__ Tn, double* __restrict__ Rn) {
  constexpr int NP = TriShape<K>::NP, NQ = TriShape<K>::NQ;
  const auto& T = tri_tab<R, K>(S);
  double s = 0.0;
#pragma unroll 4
  for (int qq = 0; qq < NQ; ++qq) s += T.psid[qq][m] * S.ts[el][qq][c];
  if (act) (c ? Rn : Tn)[(size_t)e * NP + m] = s;
}

// Split kernel: (Tn, Rn) = the projected T and rho_v of U.
template <typename R, int K, int RAIN>
__global__ void __launch_bounds__(256) tri_split_kernel(KArgs a, TriArgs t, const R* __restrict__ U,
                                                        double* __restrict__ Tn, double* __restrict__ Rn) {
  constexpr int NV = Vars<2, RAIN>::NV, NP = TriShape<K>::NP, NQ = TriShape<K>::NQ;
  constexpr int EPB = TriBlock<K>::EPB, NT = TriBlock<K>::NT, NH = (NV + 1) / 2;
  __shared__ TriLdsSplit<R, K, RAIN> S;
  const int tid = threadIdx.x;
  const bool lane = tid < NT;
  const int el = lane ? tid / NQ : 0, q = lane ? tid - el * NQ : 0;
  const int half = q >= NP ? 1 : 0, m = q - half * NP;
  const long long e0 = tri_first_element<K>(t.ne);
  if (e0 < 0) return;
  const int seen = stats_seen(a);
  const bool act = lane && e0 + el < t.ne;
  // (elements past the end repeat the last one; their results are never stored)
  const int e = (int)min(e0 + el, (long long)t.ne - 1);
  const size_t N = (size_t)t.ne * NP;
  tri_copy_tab<R, K>(S);
  if (lane) {
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const int v = half * NH + h;
      if (v < NV) S.u.cd[el][v][m] = (double)U[v * N + (size_t)e * NP + m];
    }
  }
  __syncthreads();
  int it = 0, bd = 0;
  if (lane) {
    const auto& T = tri_tab<R, K>(S);
    const TriZ g = tri_z(t, e);
    tri_split_at<R, K, RAIN>(a, S, el, q, tri_bg<K>(t, g.layer, g.z0 + g.dz1 * T.rq[q] + g.dz2 * T.sq[q]), 0.0, &it,
                             &bd);
  }
  __syncthreads();
  if (lane) tri_project_split<R, K, RAIN>(S, el, m, half, e, act, Tn, Rn);
  record_stats(a, seen, act ? it : 0, act ? bd : 0);
}

// A mode thread's share of the coefficients, and of the projected T and rho_v, of
// the neighbours across the element's faces (none on a wall).
template <typename R, int K, int RAIN>
__device__ __forceinline__ void tri_neighbours(const TriArgs& t, const R* __restrict__ U,
                                               const double* __restrict__ aux, size_t N, int e, int m, int half,
                                               bool lane, R (*nreg)[(Vars<2, RAIN>::NV + 1) / 2], double* areg) {
  constexpr int NV = Vars<2, RAIN>::NV, NH = (NV + 1) / 2, NP = TriShape<K>::NP;
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    const int nb = lane ? t.nbr[(size_t)e * 3 + f] : -1;
    const unsigned long long nm = (unsigned long long)(nb >> 2) * NP + m;
    areg[f] = 0.0;
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const int v = half * NH + h;
      nreg[f][h] = R(0);
      if (nb >= 0 && v < NV) nreg[f][h] = U[v * N + nm];
    }
    if (nb >= 0) areg[f] = aux[half * N + nm];
  }
}

// Wavefronts per SIMD that the registers are bound to.  FP32 4 (128 registers, 8
// spilled at P3; left free, 148 and 3 wavefronts: 2.12 against 1.97 ms for five
// steps), FP64 3.  With rain at P3 and P4 the LDS allows less, and a bound that it
// forbids is no bound: the compiler took 197 and more than 256 registers in FP32.
// Three steps of 200 x 100 x 2 with rain: P3 FP32 1050 -> 943 us, FP64 2008 -> 1340;
// P4 FP32 (100 x 50 x 2) 875 -> 640.  P4 in FP64 keeps one wavefront (two would
// spill 150 registers, 4.4 -> 5.3 ms).  The tendency alone (MODE 0) with rain at P3
// spills 22 and 20 registers, and is slower still with a wavefront less: 240 x 120 x
// 2 129 -> 133 us in FP32, 178 -> 230 in FP64 (230 and 413 before these bounds).
template <typename R, int K, int RAIN>
constexpr int tri_min_waves() {
  if (RAIN && K >= 3) return sizeof(R) == 4 ? (K == 4 ? 2 : 3) : (K == 4 ? 1 : 2);
  return sizeof(R) == 4 ? 4 : 3;
}

// Stage kernel.  MODE 0: out = dC/dt.  MODE 2: out = c0 U0 + c1 U + c2 dt dC/dt
// and the split of out into (Tn, Rn) for the next stage.  aux holds the
// projected T and rho_v of U: aux[0 .. N) and aux[N .. 2N), N = ne NP.
template <typename R, int K, int RAIN, int MODE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(tri_min_waves<R, K, RAIN>())))
tri_stage_kernel(KArgs a, TriArgs t, const R* __restrict__ U, const double* __restrict__ aux, R* __restrict__ out,
                 const R* __restrict__ U0, double c0, double c1, double c2dt, double* __restrict__ Tn,
                 double* __restrict__ Rn) {
  using V = Vars<2, RAIN>;
  constexpr int NV = V::NV, NP = TriShape<K>::NP, NQ = TriShape<K>::NQ, NF = TriShape<K>::NF;
  constexpr int EPB = TriBlock<K>::EPB, NT = TriBlock<K>::NT;
  constexpr int NH = (NV + 1) / 2;
  static_assert(NQ == 2 * NP, "the Duffy rule has twice as many points as P^k has modes");
  using LD = TriLds<R, K, RAIN>;
  __shared__ LD S;
  const auto& T = tri_tab<R, K>(S);
  const int tid = threadIdx.x;
  const bool lane = tid < NT;
  const int el = lane ? tid / NQ : 0, q = lane ? tid - el * NQ : 0;
  // as a mode thread: mode m; variables half NH .. (half + 1) NH of the update
  const int half = q >= NP ? 1 : 0, m = q - half * NP;
  const long long e0 = tri_first_element<K>(t.ne);
  if (e0 < 0) return;
  const int seen = MODE == 2 ? stats_seen(a) : 0;
  const bool act = lane && e0 + el < t.ne;
  // (elements past the end repeat the last one; their results are never stored)
  const int e = (int)min(e0 + el, (long long)t.ne - 1);
  const size_t N = (size_t)t.ne * NP;

  // the element's coefficients, and those of the neighbours across its faces
  // (parked in registers until the volume phase has released its LDS): thread
  // (el, m, half) takes mode m of its variables everywhere, so consecutive
  // threads read consecutive values and no index needs a division
  //
  // With rain at P3 and P4, where registers are short, what lives across the volume
  // phase is cut: the neighbours are loaded after the points (in flight during the
  // mode sums), and the split forms the background a second time (P3 FP64, three
  // steps 1851 -> 1340 us).  Elsewhere both cost time (P3 FP32 without rain 1.17 ->
  // 1.25 ms).
  constexpr bool LATE = RAIN && K >= 3;
  R nreg[3][NH];
  double areg[3];
  {
    const unsigned long long em = (unsigned long long)e * NP + m;
    if (lane) {
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        const int v = half * NH + h;
        if (v < NV) S.c[el][v][m] = U[v * N + em];
      }
      S.aux[el][half][m] = aux[half * N + em];
    }
    if constexpr (!LATE) tri_neighbours<R, K, RAIN>(t, U, aux, N, e, m, half, lane, nreg, areg);
  }
  tri_copy_tab<R, K>(S);

  // geometry: A = [V1 - V0, V2 - V0], G = A^{-T}
  const double* xv = t.xy + (size_t)e * 6;
  const TriZ g = tri_z(t, e);
  const double a00 = xv[2] - xv[0], a01 = xv[4] - xv[0], a10 = g.dz1, a11 = g.dz2;
  const double det = a00 * a11 - a01 * a10;
  const double idet = rcp64(det);
  // the face geometry, for whichever threads take the element's face points
  if (lane && q < 3) {
    const double ex = q == 0 ? a00 : (q == 1 ? a01 - a00 : -a01);
    const double ez = q == 0 ? a10 : (q == 1 ? a11 - a10 : -a11);
    const double len = sqrt(ex * ex + ez * ez);
    S.fn[el][q][0] = (R)(ez / len);
    S.fn[el][q][1] = (R)(-ex / len);
    S.fn[el][q][2] = (R)(len * idet);
    if (q == 0) S.fz[el] = g;
  }
  __syncthreads();

  // volume point q: flux along the columns of A^{-T} and sources, weighted
  Bg b{};
  if (lane) {
    R Uq[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      R s = R(0);
#pragma unroll
      for (int k = 0; k < NP; ++k) s += S.c[el][v][k] * T.psi[q][k];
      Uq[v] = s;
    }
    double Tq = 0.0, Rq = 0.0;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      Tq += S.aux[el][0][k] * T.psid[q][k];
      Rq += S.aux[el][1][k] * T.psid[q][k];
    }
    if (MODE == 2) S.ts[el][q][0] = Tq;   // the split's guess, by the same thread
    b = tri_bg<K>(t, g.layer, g.z0 + g.dz1 * T.rq[q] + g.dz2 * T.sq[q]);
    Pt<R, 2, RAIN> p;
    tri_eval<R, RAIN>(a, Uq, Tq, Rq, b, p);
    const R wq = T.w[q];
    R P[3 * NV];
    flux_dir<R, RAIN>(p, wq * (R)(a11 * idet), wq * (R)(-a01 * idet), P);
    flux_dir<R, RAIN>(p, wq * (R)(-a10 * idet), wq * (R)(a00 * idet), P + NV);
    R Gs[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) Gs[v] = R(0);
    sources<R, 2, RAIN>(a, Uq, p, Gs);
#pragma unroll
    for (int v = 0; v < NV; ++v) P[2 * NV + v] = wq * Gs[v];
#pragma unroll
    for (int v = 0; v < 3 * NV; ++v) S.u.pf[el][q * LD::PF + v] = P[v];
  }
  if constexpr (LATE) tri_neighbours<R, K, RAIN>(t, U, aux, N, e, m, half, lane, nreg, areg);
  __syncthreads();

  // modes: (F, grad psi_m) + (G, psi_m), all variables over half of the points
  R acc[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) acc[v] = R(0);
  if (lane) {
#pragma unroll 2
    for (int i = 0; i < NP; ++i) {
      const int qq = half * NP + i;
      const R* const pf = &S.u.pf[el][qq * LD::PF];
      const R dr = T.g3[qq][m][0], ds = T.g3[qq][m][1], ps = T.g3[qq][m][2];
#pragma unroll
      for (int v = 0; v < NV; ++v)
        acc[v] += pf[v] * dr + pf[NV + v] * ds + pf[2 * NV + v] * ps;
    }
    // each half leaves the partial sums that the other one finishes
#pragma unroll
    for (int v = 0; v < NV; ++v)
      if ((v >= NH) == (half == 0)) S.f.px[el][m][v] = acc[v];
  }
  __syncthreads();
  R r[NH];
  if (lane) {
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const R own = half ? (NH + h < NV ? acc[NH + h < NV ? NH + h : 0] : R(0)) : acc[h];
      r[h] = half * NH + h < NV ? own + S.f.px[el][m][half * NH + h] : R(0);
    }
#pragma unroll
    for (int f = 0; f < 3; ++f) {
#pragma unroll
      for (int h = 0; h < NH; ++h)
        if (half * NH + h < NV) S.u.nb.c[el][f][half * NH + h][m] = nreg[f][h];
      S.u.nb.aux[el][f][half][m] = areg[f];
    }
  }
  __syncthreads();

  // face point j = f NF + i of element slot fe: the Lax-Friedrichs flux
  // against the neighbour's trace (or the slip-wall ghost), weighted by
  // |e_f| / det A and w_i / 2.  The EPB 3 NF face tasks go to the block's
  // first threads, so whole wavefronts skip this phase instead of every
  // wavefront running it with idle lanes.
  static_assert(EPB * 3 * NF <= 256, "face tasks exceed the block");
  if (tid < EPB * 3 * NF) {
    const int fe = tid / (3 * NF), j = tid - fe * (3 * NF);
    const int f = j / NF, i = j - f * NF;
    const int ef = (int)min(e0 + fe, (long long)t.ne - 1);
    const TriZ gf = S.fz[fe];
    const R nx = S.fn[fe][f][0], nz = S.fn[fe][f][1];
    const int nb = t.nbr[(size_t)ef * 3 + f];
    const bool wall = nb < 0;
    const double z = gf.z0 + gf.dz1 * T.rf[f][i] + gf.dz2 * T.sf[f][i];
    const int lp_ = wall ? gf.layer : t.layer[nb >> 2];
    R Um[NV], Up[NV], Fm[NV], Fp[NV], lm, lp;
    double Tm = 0.0, Rm = 0.0;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      R s = R(0);
#pragma unroll
      for (int k = 0; k < NP; ++k) s += S.c[fe][v][k] * T.psif[f][i][k];
      Um[v] = s;
      asm volatile("" : "+v"(Um[v]));
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      Tm += S.aux[fe][0][k] * T.psifd[f][i][k];
      Rm += S.aux[fe][1][k] * T.psifd[f][i][k];
    }
    {
      Pt<R, 2, RAIN> pm;
      tri_eval<R, RAIN>(a, Um, Tm, Rm, tri_bg<K>(t, gf.layer, z), pm);
      flux_dir<R, RAIN>(pm, nx, nz, Fm);
      lm = speed_dir<R, RAIN>(pm, nx, nz);
    }
    // (the neighbour's LDS reads wait here: in flight with the own ones they
    // would need more registers than the kernel has)
    __builtin_amdgcn_sched_barrier(0);
    {
      double Tp = Tm, Rp = Rm;
      if (wall) {
        // slip wall: m+ = m- - 2 (m-.n) n, everything else copied
#pragma unroll
        for (int v = 0; v < NV; ++v) Up[v] = Um[v];
        const R mn = Um[V::M0] * nx + Um[V::M0 + 1] * nz;
        Up[V::M0] = Um[V::M0] - R(2) * mn * nx;
        Up[V::M0 + 1] = Um[V::M0 + 1] - R(2) * mn * nz;
      } else {
        // the neighbour's trace at its face point K - i (the same physical point)
        const int f2 = nb & 3, i2 = K - i;
        Tp = 0.0;
        Rp = 0.0;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          R s = R(0);
#pragma unroll
          for (int k = 0; k < NP; ++k) s += S.u.nb.c[fe][f][v][k] * T.psif[f2][i2][k];
          Up[v] = s;
          asm volatile("" : "+v"(Up[v]));
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int k = 0; k < NP; ++k) {
          Tp += S.u.nb.aux[fe][f][0][k] * T.psifd[f2][i2][k];
          Rp += S.u.nb.aux[fe][f][1][k] * T.psifd[f2][i2][k];
        }
      }
      Pt<R, 2, RAIN> pp;
      tri_eval<R, RAIN>(a, Up, Tp, Rp, tri_bg<K>(t, lp_, z), pp);
      flux_dir<R, RAIN>(pp, nx, nz, Fp);
      lp = speed_dir<R, RAIN>(pp, nx, nz);
    }
    const R L = lm >= lp ? lm : lp;
    const R wgt = S.fn[fe][f][2] * T.wf[i];
#pragma unroll
    for (int v = 0; v < NV; ++v)
      S.f.ff[fe][j * LD::NVP + v] = wgt * (R(0.5) * (Fm[v] + Fp[v]) + R(0.5) * L * (Um[v] - Up[v]));
  }
  // the mode threads' share of U0, in flight while the faces finish
  R u0[NH];
  if (MODE != 0 && c0 != 0.0 && lane) {
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const int v = half * NH + h;
      if (v < NV) u0[h] = U0[v * N + (size_t)e * NP + m];
    }
  }
  __syncthreads();

  // modes: minus the face integrals, then the update
  if (lane) {
#pragma unroll
    for (int j = 0; j < 3 * NF; ++j) {
      const R ps = T.psif[j / NF][j % NF][m];
#pragma unroll
      for (int h = 0; h < NH; ++h)
        if (half * NH + h < NV) r[h] -= S.f.ff[el][j * LD::NVP + half * NH + h] * ps;
    }
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const int v = half * NH + h;
      if (v < NV) {
        R x = r[h];
        if (MODE != 0) {
          x = (R)c1 * S.c[el][v][m] + (R)c2dt * r[h];
          if (c0 != 0.0) x += (R)c0 * u0[h];
          S.u.cd[el][v][m] = (double)x;
        }
        if (act) out[v * N + (size_t)e * NP + m] = x;
      }
    }
  }
  if constexpr (MODE == 2) {
    // the split of the updated state for the next stage (Section 3.4), from the
    // projected T of the stage input
    __syncthreads();
    int it = 0, bd = 0;
    if (lane) {
      if constexpr (LATE) {
        const TriZ z = tri_z(t, e);
        b = tri_bg<K>(t, z.layer, z.z0 + z.dz1 * T.rq[q] + z.dz2 * T.sq[q]);
      }
      tri_split_at<R, K, RAIN>(a, S, el, q, b, S.ts[el][q][0], &it, &bd);
    }
    __syncthreads();
    if (lane) tri_project_split<R, K, RAIN>(S, el, m, half, e, act, Tn, Rn);
    record_stats(a, seen, act ? it : 0, act ? bd : 0);
  }
}

// Projection onto P^k of fields given at the volume points: one thread per
// (field, element).
template <typename R, int K>
__global__ void __launch_bounds__(64) tri_project_kernel(TriArgs t, const double* __restrict__ vals, int nfields,
                                                         R* __restrict__ C) {
  constexpr int NP = TriShape<K>::NP, NQ = TriShape<K>::NQ;
  const auto& T = ttab<R, K>();
  const long long b = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= (long long)nfields * t.ne) return;
  double s[NP];
#pragma unroll
  for (int m = 0; m < NP; ++m) s[m] = 0.0;
#pragma unroll 1
  for (int q = 0; q < NQ; ++q) {
    const double wv = T.wd[q] * vals[b * NQ + q];
#pragma unroll
    for (int m = 0; m < NP; ++m) s[m] += wv * T.psid[q][m];
  }
#pragma unroll
  for (int m = 0; m < NP; ++m) C[b * NP + m] = (R)s[m];
}

// Background pressure at every layer height: the equation of state of the
// split background.
__global__ void tri_bg_pressure_kernel(KArgs a, double* bgl, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double* b = bgl + (size_t)i * 5;
  const double rd = b[0], rm = b[1], rr = a.rain ? b[2] : 0.0;
  const SplitOut s = split_point(a, rd, rm, rr, b[3], 0.0);
  const double rv = fmin(s.rvs, rm);
  b[4] = s.bad ? __builtin_nan("") : (rd * a.Rd + rv * a.Rv) * s.T;
}

}  // namespace dgm
