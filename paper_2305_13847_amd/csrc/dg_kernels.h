// Kernels of libdgmoist and their launch dispatch (instantiated per precision
// in dg_stage_f64.hip and its siblings).
//
// Work decomposition: a block owns EPB consecutive elements of one member
// (a work item); one thread owns one node of one element and computes every
// variable there (and takes face tasks; threads beyond the nodes only those).
// Elements are consecutive in x, so a block's loads are contiguous per variable.
// Q3 hexahedra have kernels of their own (dg_q3.h, dg_gauss_q3.h).
#pragma once
#include "dg_device.h"

namespace dgm {

template <int D>
struct ElemCoord {
  int c[3];
};

// Coordinates of element e0 + le of a work item (items may run past the end of
// an x-row; the carry moves to the next row).
template <int D>
__device__ __forceinline__ ElemCoord<D> item_coord(const Item& item, int le) {
  ElemCoord<D> ec;
  ec.c[0] = item.c0 + le;
  ec.c[1] = item.c12 & 0xffff;
  ec.c[2] = item.c12 >> 16;
  while (ec.c[0] >= item.n[0]) {
    ec.c[0] -= item.n[0];
    if (++ec.c[1] >= item.n[1] && D == 3) {
      ec.c[1] = 0;
      ++ec.c[2];
    }
  }
  return ec;
}

__device__ __forceinline__ int elem_stride(const Item& item, int j) {
  return j == 0 ? 1 : (j == 1 ? item.n[0] : item.n[0] * item.n[1]);
}

// Work items (member, first element) of EPB elements are dealt to blocks.
// Consecutive blocks go round-robin to the 8 XCDs; XCD x owns the contiguous
// item range [x per, (x+1) per), so neighbouring elements share an L2.  With a
// persistent grid (fewer blocks than items) each block walks its XCD's range
// with stride gridDim/8.  gridDim.x is always a multiple of 8.  A reversed
// walk (rev) runs each XCD's range from the top down: every XCD keeps its
// own items (and so what its L2 holds of them) and starts on the ones it
// wrote last.
struct ItemWalk {
  int per, g8, x, l, nitems, rev;
  __device__ __forceinline__ explicit ItemWalk(int n, int reverse = 0) {
    nitems = n;
    rev = reverse;
    per = (n + 7) >> 3;
    g8 = gridDim.x >> 3;
    x = blockIdx.x & 7;
    l = blockIdx.x >> 3;
  }
  // item of the k-th iteration, or -1 when the walk is over (uniform per block)
  __device__ __forceinline__ int item(int k) const {
    const int li = l + k * g8;
    if (li >= per) return -1;
    const int it = x * per + (rev ? per - 1 - li : li);
    return it < nitems ? it : -1;
  }
};

// Q3 hexahedra: a block is a brick of BX x BY elements (x, y), 2 x 2; meshes of
// one element along x or y throughout take 1 there.  (Half or three quarters of a
// 2 x 2 brick's wavefronts would have nothing to do, and its LDS still keeps
// others out: with rain, two steps, 1 x 1 x 8192 in FP32 298 -> 182 us, FP64
// 546 -> 266, 160 x 1 x 80 with diffusion in FP64 1375 -> 905.)  Element (dx, dy)
// of the brick is wavefront dx + BX dy.
template <int BX, int BY>
struct Brick {
  static constexpr int WPB = BX * BY;
  int dx, dy, ex, ey, ez;   // this wavefront's element: in the brick, in the mesh
  bool act, px, py;         // it exists (odd mesh sizes); its partners in x and y do
  __device__ __forceinline__ Brick(const Item& item, int w)
      : dx(BX == 2 ? w & 1 : 0),
        dy(BY == 2 ? w >> (BX - 1) : 0),
        ex(item.c0 + dx),
        ey((item.c12 & 0xffff) + dy),
        ez(item.c12 >> 16),
        act(ex < item.n[0] && ey < item.n[1]),
        px(BX == 2 && (dx == 1 || ex + 1 < item.n[0])),
        py(BY == 2 && (dy == 1 || ey + 1 < item.n[1])) {}
};

// Threads of a block of the 2D and 3D block kernels for `nodes` nodes: whole
// wavefronts; at 2D Q2, where an element has 12 face nodes to its 9 nodes, as
// many as there are face tasks (one pass instead of two).
constexpr int block_kernel_threads(int K, int D, int nodes) {
  const int tasks = K == 2 && D == 2 ? nodes / 9 * 12 : 0;
  const int n = K >= 2 && tasks > nodes ? tasks : nodes;
  return K >= 2 ? (n + 63) / 64 * 64 : n;
}

__host__ __device__ inline int grid_for_items(int nitems) { return ((nitems + 7) >> 3) << 3; }

// flags of a stage launch
constexpr int kRefreshRvs = 1;   // store a fresh rho_vs(T) evaluation (anchors later splits)
constexpr int kSponge = 2;       // the stage ends a time step: apply the sponge
// the diffusive tendency is part of the right-hand side: read from a.sip_out,
// or (Q3 hexahedra) formed by the stage kernel itself
constexpr int kSip = 4;

// One node's share of the element viscosity of Section 3.5: with quadrature
// weight w, w |u|^2 and w |u - v_r e_z|^2 (full density of rain rr, inverse
// density irho, momentum m).  sip_alpha_kernel and the Q3 stage epilogue both call this, and both
// sum the shares over the element in the same pairwise order, so alpha_K has
// the same bits whichever kernel formed it.
template <int D, int RAIN>
__device__ __forceinline__ void sip_alpha_terms(const KArgs& a, double w, double rr, double irho,
                                                const double* m, double& s0, double& s1) {
  double vr = 0.0;
  if (RAIN) vr = a.vr_mode == 0 ? a.vr_const : (rr > 0.0 ? a.vr_pref * pow(rr, 0.125) : 0.0);
  double h = 0.0;   // the horizontal part is common to both
#pragma unroll
  for (int i = 0; i < D - 1; ++i) {
    const double ui = m[i] * irho;
    h = fma(ui, ui, h);
  }
  const double uz = m[D - 1] * irho, ur = uz - vr;
  s0 = w * fma(uz, uz, h);
  s1 = w * fma(ur, ur, h);
}

// The sponge at the end of a step (Section 3.6):
// (rho_m', rho_r', m, E') <- (1 - delta) (rho_m', rho_r', m, E') with the
// far field at rest, and the moist mass removed goes to rho_d' at the node.
template <typename R, int D, int RAIN>
__device__ __forceinline__ void sponge_point(const KArgs& a, int iz, R* Un) {
  using V = Vars<D, RAIN>;
  const R dl = (R)a.sponge[iz];
  if (dl == R(0)) return;
  R lost = Un[V::RM] * dl;
  if (RAIN) lost = lost + Un[V::RR] * dl;
  const R keep = R(1) - dl;
#pragma unroll
  for (int v = 1; v < V::NV; ++v) Un[v] = Un[v] * keep;
  Un[V::RD] = Un[V::RD] + lost;
}

// ---------------------------------------------------------------------------
// split kernel: (T, rho_vs) per node, or the API outputs (T, rho_v, rho_c)
// ---------------------------------------------------------------------------
template <typename R, int K, int D, int RAIN, int API>
__global__ void __launch_bounds__(256)
split_kernel(KArgs a, int item0, int nitems, const R* __restrict__ U, const double* __restrict__ Tguess,
             double* __restrict__ oT, double* __restrict__ o1, double* __restrict__ o2) {
  using S = Shape<K, D, block_threads<R>()>;
  using V = Vars<D, RAIN>;
  constexpr int P1 = S::P1, NP = S::NP, NV = V::NV;
  // one work item per block (no item loop: loop-invariant values would stay
  // live across the body)
  const int it_ = ItemWalk(nitems).item(0);
  if (it_ < 0) return;
  const int seen = stats_seen(a);
  const int t = threadIdx.x;
  const Item item = a.items[item0 + it_];
  const MemberDesc& md = a.mem[item.member];
  const int le = t / NP, n = t - le * NP;
  const int e = item.e0 + le;
  const bool active = e < item.ne;
  int iters = 0, bad = 0;
  if (active) {
    const unsigned N = a.nnodes;
    const unsigned g = (unsigned)(item.eoff + e) * NP + n;
    const ElemCoord<D> ec = item_coord<D>(item, le);
    const int l = (D == 2) ? n / P1 : n / (P1 * P1);
    const int iz = item.hoff + ec.c[D - 1] * P1 + l;
    R Uq[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) Uq[v] = (U + (size_t)v * N)[g];
    const Bg bg = bg_at(a, iz);
    const double rd = bg.rd + (double)Uq[V::RD];
    const double rm = bg.rm + (double)Uq[V::RM];
    const double rr = RAIN ? bg.rr + (double)Uq[V::RR] : 0.0;
    const double rho = rd + rm + rr;
    double ke = 0.0;
#pragma unroll
    for (int i = 0; i < D; ++i) {
      const double mi = (double)Uq[V::M0 + i];
      ke += mi * mi;
    }
    const double re = bg.E + (double)Uq[V::E] - 0.5 * ke * rcp64(rho);
    const double guess = Tguess ? Tguess[g] : 0.0;
    const SplitOut s = split_scratch(a, rd, rm, rr, re, guess);
    iters = s.iters;
    bad = s.bad;
    oT[g] = s.T;
    if (API) {
      const double rv = fmin(s.rvs, rm);
      if (o1) o1[g] = rv;
      if (o2) o2[g] = rm - rv;
    } else {
      o1[g] = s.rvs;   // from a fresh evaluation: it anchors later splits
    }
  }
  record_stats(a, seen, iters, bad);
}

// ---------------------------------------------------------------------------
// right-hand side / stage kernel
// ---------------------------------------------------------------------------
// MODE 0: out = dU/dt
// MODE 2: out = c0 U0 + c1 U + c2 dt_member dU/dt  (a Shu-Osher stage; without
//         dt_m the time step is in c2), then the split of the new state at
//         every node, written to (oT, oS), warm-started and anchored at the
//         input state's (T, rho_vs).  With kRefreshRvs the stored rho_vs is a
//         fresh evaluation at the new T, otherwise the anchored one.  With
//         kSponge the new state is the end of a step: the sponge acts on it
//         before it is stored and split.
template <typename R, int D, int RAIN>
struct Nb {
  R U[Vars<D, RAIN>::NV];
  double T, rvs;
};

template <typename R, int K, int D, int RAIN, int J>
__device__ __forceinline__ void gather_nb(const Item& item, const ElemCoord<D>& ec, int e, int n,
                                          int ij, const R* __restrict__ U,
                                          const double* __restrict__ auxT,
                                          const double* __restrict__ auxS, unsigned N,
                                          Nb<R, D, RAIN>& nb, bool& wall, int& izn_off) {
  using S = Shape<K, D, block_threads<R>()>;
  using V = Vars<D, RAIN>;
  constexpr int P1 = S::P1, NV = V::NV;
  constexpr int STR = (J == 0) ? 1 : (J == 1 ? P1 : P1 * P1);
  const bool plus = (ij == K);
  const int c = ec.c[J];
  const bool at_end = plus ? (c == item.n[J] - 1) : (c == 0);
  wall = at_end && item.bc[J] == 1;
  if (wall) return;
  int cn = plus ? c + 1 : c - 1;
  if (cn < 0) cn += item.n[J];
  if (cn >= item.n[J]) cn -= item.n[J];
  const int en = e + (cn - c) * elem_stride(item, J);
  const int nn = plus ? n - K * STR : n + K * STR;
  const unsigned gn = (unsigned)(item.eoff + en) * S::NP + nn;
#pragma unroll
  for (int v = 0; v < NV; ++v) nb.U[v] = (U + (size_t)v * N)[gn];
  nb.T = auxT[gn];
  nb.rvs = auxS[gn];
  izn_off = (J == D - 1) ? (cn * P1 + (plus ? 0 : K)) : -1;
}

// Volume term (Section 3.2 weak form, Lobatto collocation): for direction J,
// R += (2/h_J) sum_b Dhat[i_J][b] F_J(node b on this node's J-line).  The
// fluxes of all directions are staged in LDS behind one barrier.
template <typename R, int K, int D, int RAIN, int J>
__device__ __forceinline__ void volume_dir(const MemberDesc& md, int ij, const R* sFJ, R* Rv,
                                           const R* sD, int t = threadIdx.x) {
  using S = Shape<K, D, block_threads<R>()>;
  using V = Vars<D, RAIN>;
  constexpr int P1 = S::P1, NV = V::NV;
  constexpr int STR = (J == 0) ? 1 : (J == 1 ? P1 : P1 * P1);
    constexpr int NT = S::NT;   // LDS row stride (the largest block)
  const R s = (R)md.two_over_h[J];
  const int base = t - ij * STR;
  R d[P1];
#pragma unroll
  for (int b = 0; b < P1; ++b) d[b] = sD[ij * P1 + b];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    R acc = R(0);
#pragma unroll
    for (int b = 0; b < P1; ++b) acc += d[b] * sFJ[v * NT + base + b * STR];
    Rv[v] += s * acc;
  }
}

// The three directions of volume_dir, variable by variable: the scheduling
// barrier keeps the compiler from issuing the LDS reads of every variable at
// once (their results would need more registers than the kernel has).
template <typename R, int K, int RAIN>
__device__ __forceinline__ void volume_3d(const MemberDesc& md, const int* idx, const R* sF, R* Rv, const R* sD,
                                          int t) {
  using S = Shape<K, 3, block_threads<R>()>;
  constexpr int P1 = S::P1, NV = Vars<3, RAIN>::NV, NT = S::NT;
  R s[3], d[3][P1];
  int base[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int str = j == 0 ? 1 : (j == 1 ? P1 : P1 * P1);
    s[j] = (R)md.two_over_h[j];
    base[j] = j * (NV * NT) + t - idx[j] * str;
#pragma unroll
    for (int b = 0; b < P1; ++b) d[j][b] = sD[idx[j] * P1 + b];
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int str = j == 0 ? 1 : (j == 1 ? P1 : P1 * P1);
      R acc = R(0);
#pragma unroll
      for (int b = 0; b < P1; ++b) acc += d[j][b] * sF[v * NT + base[j] + b * str];
      Rv[v] += s[j] * acc;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <typename R, int K, int D, int RAIN, int J>
__device__ __forceinline__ void stage_flux(const Pt<R, D, RAIN>& q, R* sFJ) {
  using V = Vars<D, RAIN>;
  constexpr int NV = V::NV;
  constexpr int NT = Shape<K, D, block_threads<R>()>::NT;   // LDS row stride (the largest block)
  R F[NV];
  flux<R, D, RAIN, J>(q, F);
#pragma unroll
  for (int v = 0; v < NV; ++v) sFJ[v * NT + threadIdx.x] = F[v];
}

template <typename R, int K, int D, int RAIN, int J>
__device__ __forceinline__ void face_dir(const KArgs& a, const Item& item, const MemberDesc& md, int ij, int iz,
                                         const R* Uq, const Pt<R, D, RAIN>& q, const Nb<R, D, RAIN>& nb,
                                         bool wall, int izn_off, R* Rv) {
  using V = Vars<D, RAIN>;
  constexpr int NV = V::NV;
  const bool plus = (ij == K);
  R Un[NV];
  Pt<R, D, RAIN> qn;
  if (wall) {
#pragma unroll
    for (int v = 0; v < NV; ++v) Un[v] = Uq[v];
    Un[V::M0 + J] = -Uq[V::M0 + J];
    qn = q;
    reflect<R, D, RAIN, J>(qn);
  } else {
#pragma unroll
    for (int v = 0; v < NV; ++v) Un[v] = nb.U[v];
    const int izn = (J == D - 1) ? item.hoff + izn_off : iz;
    eval_point<R, D, RAIN>(a, Un, nb.T, nb.rvs, izn, qn);
  }
  R F[NV], Fn[NV];
  flux<R, D, RAIN, J>(q, F);
  flux<R, D, RAIN, J>(qn, Fn);
  const R lo = wave_speed<R, D, RAIN, J>(q);
  const R ln = wave_speed<R, D, RAIN, J>(qn);
  // Lambda = max over the two sides, ties to the minus side
  const R Lam = plus ? ((lo >= ln) ? lo : ln) : ((ln >= lo) ? ln : lo);
  const R half = R(0.5);
  if (plus) {
    const R lift = (R)md.lift[J][1];
#pragma unroll
    for (int v = 0; v < NV; ++v) Rv[v] -= lift * (half * (F[v] + Fn[v]) + half * Lam * (Uq[v] - Un[v]));
  } else {
    const R lift = (R)md.lift[J][0];
#pragma unroll
    for (int v = 0; v < NV; ++v) Rv[v] += lift * (half * (Fn[v] + F[v]) + half * Lam * (Un[v] - Uq[v]));
  }
}

// Face work of a block: the epb 2 D (K+1)^(D-1) (direction, element, side, face
// node) tasks in that order, one per lane, taken by all of the block's
// wavefronts in turn, so a lane's direction is a run-time value.  (One
// direction per wavefront, as before, left the remainder of every direction
// idle and a block's last, partly filled wavefront out: with 125 threads all
// face work ran on one wavefront.)
template <int K, int D>
struct FaceShape {
  static constexpr int P1 = K + 1;
  static constexpr int FN = (D == 2) ? P1 : P1 * P1;  // nodes per face
  static constexpr int NP = Shape<K, D>::NP;
};

// Per element of the block (3D): the first height index, the matching height
// index of the vertical neighbours below and above, and per (direction, side)
// the neighbour's first node (kWall: a slip wall, kNone: no element).  Formed
// once per block by one thread per element and face; the nodes and the face
// tasks read it.
//
// On a slip wall the neighbour of a face node is its own mirror image: the
// task reads the own node and reverses the normal momentum.
constexpr unsigned kWall = 0xffffffffu, kNone = 0xfffffffeu;
template <int D>
struct ElemTab {
  int iz, izn[2];
  unsigned nb[2 * D];
};

template <int K, int D>
__device__ __forceinline__ void elem_table(const Item& item, int epb, int t, ElemTab<D>* tab) {
  constexpr int P1 = K + 1, NP = FaceShape<K, D>::NP;
  if (t >= epb * 2 * D) return;
  const int le = t / (2 * D), f = t - le * (2 * D);
  const int j = f >> 1, side = f & 1;
  const int e = item.e0 + le;
  if (e >= item.ne) {
    tab[le].nb[f] = kNone;
    return;
  }
  const ElemCoord<D> ec = item_coord<D>(item, le);
  const int c = j == 0 ? ec.c[0] : (j == 1 ? ec.c[1] : ec.c[2]);
  // (copies in scalar registers: a select of array elements would put the item
  // into scratch memory)
  int ns[3], bs[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    ns[k] = __builtin_amdgcn_readfirstlane(item.n[k]);
    bs[k] = __builtin_amdgcn_readfirstlane(item.bc[k]);
  }
  const int n = j == 0 ? ns[0] : (j == 1 ? ns[1] : ns[2]);
  const int bc = j == 0 ? bs[0] : (j == 1 ? bs[1] : bs[2]);
  const int st = j == 0 ? 1 : (j == 1 ? ns[0] : ns[0] * ns[1]);
  const bool at_end = side ? c == n - 1 : c == 0;
  const int step = at_end ? (side ? 1 - n : n - 1) : (side ? 1 : -1);
  tab[le].nb[f] = at_end && bc == 1 ? kWall : (unsigned)(item.eoff + e + step * st) * NP;
  if (j == D - 1) tab[le].izn[side] = item.hoff + (c + step) * P1 + (side ? 0 : K);
  if (f == 0) tab[le].iz = item.hoff + ec.c[D - 1] * P1;
}

// Physical flux in a direction chosen per lane.
template <typename R, int D, int RAIN>
__device__ __forceinline__ void flux_sel(const Pt<R, D, RAIN>& q, int J, R uj, R* F) {
  using V = Vars<D, RAIN>;
  const bool vert = J == D - 1;
  const R fall = RAIN && vert ? q.rrvr : R(0);
  F[V::RD] = q.rd * uj;
  F[V::RM] = q.rm * uj;
  if (RAIN) F[V::RR] = q.rr * uj - fall;
#pragma unroll
  for (int i = 0; i < D; ++i) {
    R f = q.m[i] * uj + (i == J ? q.pp : R(0));
    if (RAIN) f -= fall * q.u[i];
    F[V::M0 + i] = f;
  }
  F[V::E] = RAIN ? q.H * uj - (vert ? q.rain_e : R(0)) : q.H * uj;
}

template <typename R, int D, int RAIN>
struct Pair {
  Nb<R, D, RAIN> nb;
  int slot;   // block slot (le * NP + n) of the own node; -1: nothing to do
  int J, side, izn;
  bool wall;
};

// own node of face node (fa, fb) of side `side` in direction J, and the step
// to the matching node of the neighbour's element
template <int K, int D>
__device__ __forceinline__ int face_node(int J, int side, int fa, int fb, int& match) {
  constexpr int P1 = K + 1;
  const int str = J == 0 ? 1 : (D == 2 || J == 1 ? P1 : P1 * P1);
  match = side ? -K * str : K * str;
  return side * K * str + fa * (J == 0 ? P1 : 1) + (D == 3 ? fb * (J == 2 ? P1 : P1 * P1) : 0);
}

template <typename R, int D, int RAIN>
__device__ __forceinline__ void pair_load(const R* __restrict__ U, const double* __restrict__ auxT,
                                          const double* __restrict__ auxS, unsigned N, unsigned gn,
                                          Pair<R, D, RAIN>& pr) {
#pragma unroll
  for (int v = 0; v < Vars<D, RAIN>::NV; ++v) pr.nb.U[v] = ld(U, N, v, gn);
  pr.nb.T = ld_f64<R>(auxT, N, gn);
  pr.nb.rvs = ld_f64<R>(auxS, N, gn);
}

// 3D task q (direction, element, side, face node): the own node, and the
// neighbour's trace.  g0: the block's first node.
template <typename R, int K, int RAIN>
__device__ __forceinline__ void pair_gather(const ElemTab<3>* tab, unsigned g0, int q, int pj, const R* __restrict__ U,
                                            const double* __restrict__ auxT, const double* __restrict__ auxS,
                                            unsigned N, Pair<R, 3, RAIN>& pr) {
  using FS = FaceShape<K, 3>;
  constexpr int P1 = FS::P1, FN = FS::FN, NP = FS::NP;
  pr.slot = -1;
  if (q >= 3 * pj) return;
  const int J = (q >= pj ? 1 : 0) + (q >= 2 * pj ? 1 : 0);
  const int rq = q - J * pj;
  const int le = rq / (2 * FN);
  const int r = rq - le * (2 * FN);
  const int side = r >= FN ? 1 : 0;
  const int f = r - side * FN;
  const unsigned nb = tab[le].nb[2 * J + side];
  if (nb == kNone) return;
  const int fb = f / P1, fa = f - fb * P1;
  int match;
  const int n = face_node<K, 3>(J, side, fa, fb, match);
  pr.wall = nb == kWall;
  pr.slot = le * NP + n;
  pr.J = J;
  pr.side = side;
  pair_load<R, 3, RAIN>(U, auxT, auxS, N, pr.wall ? g0 + (unsigned)pr.slot : nb + (unsigned)(n + match), pr);
  pr.izn = J == 2 ? (pr.wall ? tab[le].iz + side * K : tab[le].izn[side]) : tab[le].iz + fb;
}

// The neighbour's side of a pair: its normal flux Fn and wave speed; on a wall
// the mirrored state.
template <typename R, int D, int RAIN>
__device__ __forceinline__ void pair_eval(const KArgs& a, Pair<R, D, RAIN>& pr, R* Fn, R& ln) {
  using V = Vars<D, RAIN>;
  const int J = pr.J;
#pragma unroll
  for (int i = 0; i < D; ++i) pr.nb.U[V::M0 + i] = pr.wall && i == J ? -pr.nb.U[V::M0 + i] : pr.nb.U[V::M0 + i];
  Pt<R, D, RAIN> qn;
  eval_point<R, D, RAIN>(a, pr.nb.U, pr.nb.T, pr.nb.rvs, pr.izn, qn);
  const R uj = J == 0 ? qn.u[0] : (D == 3 && J == 1 ? qn.u[1] : qn.u[D - 1]);
  flux_sel<R, D, RAIN>(qn, J, uj, Fn);
  ln = fabs(uj) + qn.cm;
  if (RAIN) ln += J == D - 1 ? fabs(qn.vr) : R(0);
}

// Lax-Friedrichs flux of one pair (Section 3.2): the own trace (U, F_J,
// lambda_J) comes from the block's LDS tiles.  The lifted correction
// +-(lift/2)(F + F_n) + (lift/2) Lambda (U_n - U), + on the minus face, goes to
// out[v * stride].
template <typename R, int K, int D, int RAIN>
__device__ __forceinline__ void pair_flux(const MemberDesc& md, const Pair<R, D, RAIN>& pr, const R* Fn, R ln,
                                          const R* sF, const R* sU, const R* sL, R* out, int stride) {
  using V = Vars<D, RAIN>;
  constexpr int NV = V::NV;
  constexpr int NT = Shape<K, D, block_threads<R>()>::NT;
  const int J = pr.J;
  const R* F = sF + J * (NV * NT) + pr.slot;
  const R* Uo = sU + pr.slot;
  const R lo = sL[J * NT + pr.slot];
  // Lambda = max over the two sides, ties to the minus side
  const bool own = pr.side ? (lo >= ln) : !(ln >= lo);
  const R Lam = own ? lo : ln;
  // (the Lobatto weights are symmetric: both sides lift alike)
  const R lift = (R)(J == 0 ? md.lift[0][0] : (D == 3 && J == 1 ? md.lift[1][0] : md.lift[D - 1][0]));
  const R hl = R(0.5) * lift;
  const R kf = pr.side ? -hl : hl;
  const R kj = hl * Lam;
#pragma unroll
  for (int v = 0; v < NV; ++v) out[v * stride] = fma(kf, F[v * NT] + Fn[v], kj * (pr.nb.U[v] - Uo[v * NT]));
}

// Stage update and the split epilogue shared by both face schemes.
template <typename R, int D, int RAIN, int MODE>
__device__ __forceinline__ void stage_epilogue(const KArgs& a, const Bg& bg, int iz, unsigned g, unsigned N,
                                               const R* Uq, const R* U0q, const R* Rv, double T, double rvs,
                                               R* __restrict__ out, double dtm, double c0, double c1,
                                               double c2, double* __restrict__ oT,
                                               double* __restrict__ oS, int flags, int& iters, int& bad,
                                               R* Unew = nullptr, double* Tnew = nullptr,
                                               double* Snew = nullptr, double wq = 0.0,
                                               double* alpha_terms = nullptr) {
  // (Unew, Tnew, Snew), when given, receive the stored new state and its
  // stored (T, rho_vs); alpha_terms, when given, the node's
  // shares of the new state's element viscosity (weight wq)
  using V = Vars<D, RAIN>;
  constexpr int NV = V::NV;
  if (MODE == 0) {
#pragma unroll
    for (int v = 0; v < NV; ++v) st(out, N, v, g, Rv[v]);
    return;
  }
  const R k2 = (R)(c2 * dtm);
  const R k1 = (R)c1;
  R Un[NV];
  if (c0 != 0.0) {
    const R k0 = (R)c0;
#pragma unroll
    for (int v = 0; v < NV; ++v) Un[v] = k0 * U0q[v] + k1 * Uq[v] + k2 * Rv[v];
  } else {
#pragma unroll
    for (int v = 0; v < NV; ++v) Un[v] = k1 * Uq[v] + k2 * Rv[v];
  }
  if (flags & kSponge) sponge_point<R, D, RAIN>(a, iz, Un);
#pragma unroll
  for (int v = 0; v < NV; ++v) st(out, N, v, g, Un[v]);
  if (alpha_terms) {
    double m[D];
#pragma unroll
    for (int i = 0; i < D; ++i) m[i] = (double)Un[V::M0 + i];
    const double rr = RAIN ? bg.rr + (double)Un[V::RR] : 0.0;
    const double irho = rcp64((bg.rd + (double)Un[V::RD]) + (bg.rm + (double)Un[V::RM]) + rr);
    sip_alpha_terms<D, RAIN>(a, wq, rr, irho, m, alpha_terms[0], alpha_terms[1]);
  }
  if (Unew) {
#pragma unroll
    for (int v = 0; v < NV; ++v) Unew[v] = Un[v];
  }
  if (MODE == 2) {
    // split of the new state (FP64), warm-started at this node's (T, rho_vs);
    // bg: the background at this node
    const double rd = bg.rd + (double)Un[V::RD];
    const double rm = bg.rm + (double)Un[V::RM];
    const double rr = RAIN ? bg.rr + (double)Un[V::RR] : 0.0;
    double ke = 0.0;
#pragma unroll
    for (int i = 0; i < D; ++i) {
      const double mi = (double)Un[V::M0 + i];
      ke += mi * mi;
    }
    const double re = bg.E + (double)Un[V::E] - 0.5 * ke * rcp64(rd + rm + rr);
    const SplitOut s = split_warm<D>(a, rd, rm, rr, re, T, rvs);
    iters = s.iters;
    bad = s.bad;
    const double rvs_st = ((flags & kRefreshRvs) && s.bad == 0) ? rho_vs(a, s.T) : s.rvs;
    st_f64<R>(oT, N, g, s.T);
    st_f64<R>(oS, N, g, rvs_st);
    if (Tnew) *Tnew = s.T;
    if (Snew) *Snew = rvs_st;
  }
}

// 3D right-hand side / stage of one work item with the lane-dense face pass
// (three steps on 45 x 37 x 21 Q2, FP32: 582 -> 491 us against one direction
// per wavefront and integer decoding of the element in every pass)
// (K >= 2, where a node lies on at most one face per direction).  LDS tiles
// use the compile-time stride NT of the largest block; smaller blocks use a
// prefix of each row.  The block has whole wavefronts: threads from a.epb NP
// on own no node and take face tasks only.
template <typename R, int K, int RAIN, int MODE>
__device__ __forceinline__ void rhs_item_3d(const KArgs& a, int t, int it_, ElemTab<3>* tab, R* sF, R* sU, R* sL,
                                               const R* sD, const R* __restrict__ U,
                                               const double* __restrict__ auxT,
                                               const double* __restrict__ auxS, R* __restrict__ out,
                                               const R* __restrict__ U0, const double* __restrict__ dt_m,
                                               double c0, double c1, double c2, double* __restrict__ oT,
                                               double* __restrict__ oS, int flags) {
  constexpr int D = 3;
  using S = Shape<K, D, block_threads<R>()>;
  using V = Vars<D, RAIN>;
  using FS = FaceShape<K, D>;
  constexpr int P1 = S::P1, NP = S::NP, NV = V::NV, NT = S::NT;
  static_assert(K >= 2, "pair face pass needs K >= 2");
  const int seen = MODE == 2 ? stats_seen(a) : 0;
  const Item item = a.items[it_];
  const MemberDesc& md = a.mem[item.member];
  const int epb = a.epb;
  const unsigned N = a.nnodes;
  // the block's nodes are contiguous
  const unsigned g = (unsigned)(item.eoff + item.e0) * NP + t;
  const bool active = t < min(epb, item.ne - item.e0) * NP;
  R Uq[NV];
  double T = 300.0, rvs = 0.0;
  if (active) {
#pragma unroll
    for (int v = 0; v < NV; ++v) Uq[v] = ld(U, N, v, g);
    T = ld_f64<R>(auxT, N, g);
    rvs = ld_f64<R>(auxS, N, g);
  } else {
#pragma unroll
    for (int v = 0; v < NV; ++v) Uq[v] = R(0);
  }
  elem_table<K, D>(item, epb, t, tab);
  const double dtm = MODE != 0 && dt_m ? dt_m[item.member] : 1.0;
  const int le = t / NP, n = t - le * NP;
  int idx[3];
  idx[0] = n % P1;
  idx[1] = (n / P1) % P1;
  idx[2] = n / (P1 * P1);
  __syncthreads();   // the table (and sD)
  const int iz = active ? tab[le].iz + idx[D - 1] : item.hoff;
  const int pj = epb * 2 * FS::FN;
  R Rv[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) Rv[v] = R(0);
  if (active) {
    Pt<R, D, RAIN> q;
    eval_point<R, D, RAIN>(a, Uq, T, rvs, iz, q);
    R F[NV];
    flux<R, D, RAIN, 0>(q, F);
#pragma unroll
    for (int v = 0; v < NV; ++v) sF[v * NT + t] = F[v];
    flux<R, D, RAIN, 1>(q, F);
#pragma unroll
    for (int v = 0; v < NV; ++v) sF[(NV + v) * NT + t] = F[v];
    flux<R, D, RAIN, 2>(q, F);
#pragma unroll
    for (int v = 0; v < NV; ++v) sF[(2 * NV + v) * NT + t] = F[v];
#pragma unroll
    for (int v = 0; v < NV; ++v) sU[v * NT + t] = Uq[v];
    sL[t] = wave_speed<R, D, RAIN, 0>(q);
    sL[NT + t] = wave_speed<R, D, RAIN, 1>(q);
    sL[2 * NT + t] = wave_speed<R, D, RAIN, 2>(q);
    sources<R, D, RAIN>(a, Uq, q, Rv);
  }
  __syncthreads();
  R U0q[NV];
  Bg bg{};
  if (active) {
    volume_3d<R, K, RAIN>(md, idx, sF, Rv, sD, t);
  }
  __syncthreads();   // the volume term has read sF
  // face passes: every task runs the same code, so the rounding of a face
  // flux does not depend on the pass (the launch geometry) that computes it
#pragma clang loop unroll(disable)
  for (int k = t; k < D * pj; k += (int)blockDim.x) {
    Pair<R, D, RAIN> pr;
    pair_gather<R, K, RAIN>(tab, g - (unsigned)t, k, pj, U, auxT, auxS, N, pr);
    if (pr.slot >= 0) {
      R Fn[NV], ln;
      pair_eval<R, D, RAIN>(a, pr, Fn, ln);
      // the correction replaces F_J at the own slot
      pair_flux<R, K, D, RAIN>(md, pr, Fn, ln, sF, sU, sL, sF + pr.J * (NV * NT) + pr.slot, NT);
    }
  }
  // operands of the stage update and the split, fetched while the faces of
  // the other wavefronts finish
  if (MODE != 0 && active && c0 != 0.0) {
#pragma unroll
    for (int v = 0; v < NV; ++v) U0q[v] = ld(U0, N, v, g);
  }
  if (MODE == 2 && active) {
    bg = bg_at(a, iz);
  }
  __syncthreads();
  int iters = 0, bad = 0;
  if (active) {
#pragma unroll
    for (int j = 0; j < D; ++j)
      if (idx[j] == 0 || idx[j] == K) {
#pragma unroll
        for (int v = 0; v < NV; ++v) Rv[v] += sF[(j * NV + v) * NT + t];
      }
    R Us[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) Us[v] = sU[v * NT + t];
    if (flags & kSip) {
#pragma unroll
      for (int v = 0; v < NV; ++v) Rv[v] += ld((const R*)a.sip_out, N, v, g);
    }
    stage_epilogue<R, D, RAIN, MODE>(a, bg, iz, g, N, Us, U0q, Rv, T, rvs, out, dtm, c0, c1, c2, oT, oS, flags,
                                     iters, bad);
  }
  if (MODE == 2) record_stats(a, seen, iters, bad);
}

// 2D right-hand side / stage of one work item (K >= 2).  A 2D element has
// about as many face nodes (4 (K+1)) as nodes, so a block's face tasks are one
// pass of its threads (a loop over further ones, which no shape has, cost 2 to 10 %
// in registers and code); they are numbered element by element, and every load of
// a thread (its node, the neighbour's trace of its task, both backgrounds) is issued
// before any arithmetic: the state is read in one round trip, and nothing waits for
// memory between the barriers.
//
// Small calls are one wavefront's chain of dependent instructions, large ones
// are bound by VALU issue; with the self-contained work items and without the loop,
// ten steps on 16 x 16 Q2 (FP64) 405 -> 240 us, 128 x 64 Q4 (FP64) 482 -> 428 us; with
// the items, five of a 64-member Q3 ensemble (FP32) 3.01 -> 2.83 ms.
//
// In FP32 the corrections have an LDS tile of their own (SEP), so the faces
// need not wait for the volume term; in FP64 that tile would cost a quarter
// of the resident blocks, and they replace F_J at the own slot behind one
// more barrier.
template <typename R, int K, int RAIN>
struct Lds2d {
  using S = Shape<K, 2, block_threads<R>()>;
  static constexpr int NV = Vars<2, RAIN>::NV;
  static constexpr bool SEP = sizeof(R) == 4;
  static constexpr int NQ = S::EPB * 4 * S::P1;   // face tasks of the largest block
};

// Task q: element le = q / (4 P1), then direction, side, face node.
template <typename R, int K, int RAIN>
__device__ __forceinline__ void pair_gather_2d(const Item& item, unsigned g0, int q,
                                               const R* __restrict__ U, const double* __restrict__ auxT,
                                               const double* __restrict__ auxS, unsigned N, Pair<R, 2, RAIN>& pr) {
  constexpr int P1 = K + 1, NP = P1 * P1;
  const int le = q / (4 * P1);
  const int r = q - le * (4 * P1);
  const int J = r >= 2 * P1 ? 1 : 0;
  const int side = (J ? r - 2 * P1 : r) >= P1 ? 1 : 0;
  const int f = r - (2 * J + side) * P1;
  const ElemCoord<2> ec = item_coord<2>(item, le);
  const int c = J ? ec.c[1] : ec.c[0], nJ = J ? item.n[1] : item.n[0];
  const bool at_end = side ? c == nJ - 1 : c == 0;
  const int step = at_end ? (side ? 1 - nJ : nJ - 1) : (side ? 1 : -1);
  int match;
  const int n = face_node<K, 2>(J, side, f, 0, match);
  pr.wall = at_end && (J ? item.bc[1] : item.bc[0]) == 1;
  pr.slot = le * NP + n;
  pr.J = J;
  pr.side = side;
  const int off = pr.wall ? 0 : step * (J ? item.n[0] : 1) * NP + match;
  pair_load<R, 2, RAIN>(U, auxT, auxS, N, g0 + (unsigned)(pr.slot + off), pr);
  const int row = J && !pr.wall ? c + step : ec.c[1];
  pr.izn = item.hoff + row * P1 + (J ? ((side != 0) == pr.wall ? K : 0) : f);
}

template <typename R, int K, int RAIN, int MODE>
__device__ __forceinline__ void rhs_item_2d(const KArgs& a, int t, int it_, R* sF, R* sU, R* sL, R* sC, const R* sD,
                                            const R* __restrict__ U, const double* __restrict__ auxT,
                                            const double* __restrict__ auxS, R* __restrict__ out,
                                            const R* __restrict__ U0, const double* __restrict__ dt_m, double c0,
                                            double c1, double c2, double* __restrict__ oT, double* __restrict__ oS,
                                            int flags) {
  constexpr int D = 2;
  using S = Shape<K, D, block_threads<R>()>;
  using V = Vars<D, RAIN>;
  using L = Lds2d<R, K, RAIN>;
  constexpr int P1 = S::P1, NP = S::NP, NV = V::NV, NT = S::NT, NQ = L::NQ;
  const int seen = MODE == 2 ? stats_seen(a) : 0;
  const Item item = a.items[it_];
  const MemberDesc& md = a.mem[item.member];
  const unsigned N = a.nnodes;
  const int nel = min(a.epb, item.ne - item.e0);   // elements of this item
  const unsigned g0 = (unsigned)(item.eoff + item.e0) * NP, g = g0 + (unsigned)t;
  const bool active = t < nel * NP;
  const int ntask = nel * 4 * P1;   // at most one a thread
  static_assert(K == 2 || 4 * P1 <= NP, "an element's face tasks fit its threads (K = 2: block_kernel_threads)");
  R Uq[NV];
  double T = 300.0, rvs = 0.0;
  Pair<R, D, RAIN> pr;
  const int le = t / NP, n = t - le * NP;
  const int idx[2] = {n % P1, n / P1};
  int iz = item.hoff;
  if (active) {
#pragma unroll
    for (int v = 0; v < NV; ++v) Uq[v] = ld(U, N, v, g);
    T = ld_f64<R>(auxT, N, g);
    rvs = ld_f64<R>(auxS, N, g);
    iz = item.hoff + item_coord<D>(item, le).c[1] * P1 + idx[1];
  } else {
#pragma unroll
    for (int v = 0; v < NV; ++v) Uq[v] = R(0);
  }
  const bool task = t < ntask;
  if (task) pair_gather_2d<R, K, RAIN>(item, g0, t, U, auxT, auxS, N, pr);
  const double dtm = MODE != 0 && dt_m ? dt_m[item.member] : 1.0;
  R Rv[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) Rv[v] = R(0);
  if (active) {
    Pt<R, D, RAIN> q;
    eval_point<R, D, RAIN>(a, Uq, T, rvs, iz, q);
    R F[NV];
    flux<R, D, RAIN, 0>(q, F);
#pragma unroll
    for (int v = 0; v < NV; ++v) sF[v * NT + t] = F[v];
    flux<R, D, RAIN, 1>(q, F);
#pragma unroll
    for (int v = 0; v < NV; ++v) sF[(NV + v) * NT + t] = F[v];
#pragma unroll
    for (int v = 0; v < NV; ++v) sU[v * NT + t] = Uq[v];
    sL[t] = wave_speed<R, D, RAIN, 0>(q);
    sL[NT + t] = wave_speed<R, D, RAIN, 1>(q);
    sources<R, D, RAIN>(a, Uq, q, Rv);
  }
  R Fn[NV], ln;
  if (task) pair_eval<R, D, RAIN>(a, pr, Fn, ln);
  __syncthreads();
  auto dest = [&](int q, const Pair<R, D, RAIN>& p) { return L::SEP ? sC + q : sF + p.J * (NV * NT) + p.slot; };
  constexpr int dst = L::SEP ? NQ : NT;
  if (L::SEP && task) pair_flux<R, K, D, RAIN>(md, pr, Fn, ln, sF, sU, sL, dest(t, pr), dst);
  if (active) {
    volume_dir<R, K, D, RAIN, 0>(md, idx[0], sF, Rv, sD, t);
    volume_dir<R, K, D, RAIN, 1>(md, idx[1], sF + NV * NT, Rv, sD, t);
  }
  if (!L::SEP) {
    __syncthreads();   // the volume term has read sF
    if (task) pair_flux<R, K, D, RAIN>(md, pr, Fn, ln, sF, sU, sL, dest(t, pr), dst);
  }
  // operands of the stage update and the split, fetched while the faces of
  // the other wavefronts finish
  R U0q[NV];
  Bg bg{};
  if (MODE != 0 && active && c0 != 0.0) {
#pragma unroll
    for (int v = 0; v < NV; ++v) U0q[v] = ld(U0, N, v, g);
  }
  if (MODE == 2 && active) {
    bg = bg_at(a, iz);
  }
  __syncthreads();
  int iters = 0, bad = 0;
  if (active) {
#pragma unroll
    for (int j = 0; j < D; ++j)
      if (idx[j] == 0 || idx[j] == K) {
        const R* C = L::SEP ? sC + le * (4 * P1) + (2 * j + (idx[j] == K ? 1 : 0)) * P1 + idx[1 - j]
                            : sF + j * (NV * NT) + t;
#pragma unroll
        for (int v = 0; v < NV; ++v) Rv[v] += C[v * dst];
      }
    R Us[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) Us[v] = sU[v * NT + t];
    if (flags & kSip) {
#pragma unroll
      for (int v = 0; v < NV; ++v) Rv[v] += ld((const R*)a.sip_out, N, v, g);
    }
    stage_epilogue<R, D, RAIN, MODE>(a, bg, iz, g, N, Us, U0q, Rv, T, rvs, out, dtm, c0, c1, c2, oT, oS, flags,
                                     iters, bad);
  }
  if (MODE == 2) record_stats(a, seen, iters, bad);
}

template <typename R, int K, int D, int RAIN, int MODE>
__device__ __forceinline__ void rhs_item(const KArgs& a, int t, int it_, R (*sF)[Vars<D, RAIN>::NV * Shape<K, D, block_threads<R>()>::NT],
                                         const R* sD, const R* __restrict__ U,
                                         const double* __restrict__ auxT,
                                         const double* __restrict__ auxS, R* __restrict__ out,
                                         const R* __restrict__ U0, const double* __restrict__ dt_m,
                                         double c0, double c1, double c2, double* __restrict__ oT,
                                         double* __restrict__ oS, int flags) {
  using S = Shape<K, D, block_threads<R>()>;
  using V = Vars<D, RAIN>;
  constexpr int P1 = S::P1, NP = S::NP, NV = V::NV;
  const int seen = MODE == 2 ? stats_seen(a) : 0;
  const Item item = a.items[it_];
  const MemberDesc& md = a.mem[item.member];
  const int le = t / NP, n = t - le * NP;
  const int e = item.e0 + le;
  const bool active = e < item.ne;
  const unsigned N = a.nnodes;
  const unsigned g = (unsigned)(item.eoff + (active ? e : 0)) * NP + n;
  const ElemCoord<D> ec = item_coord<D>(item, active ? le : 0);
  int idx[3];
  idx[0] = n % P1;
  idx[1] = (n / P1) % P1;
  idx[2] = (D == 3) ? n / (P1 * P1) : 0;
  const int iz = item.hoff + ec.c[D - 1] * P1 + idx[D - 1];
  R Uq[NV];
  double T = 300.0, rvs = 0.0;
  if (active) {
#pragma unroll
    for (int v = 0; v < NV; ++v) Uq[v] = (U + (size_t)v * N)[g];
    T = auxT[g];
    rvs = auxS[g];
  } else {
#pragma unroll
    for (int v = 0; v < NV; ++v) Uq[v] = R(0);
  }
  // neighbour traces: issue every gather before any arithmetic
  Nb<R, D, RAIN> nb0, nb1, nb2;
  bool w0 = false, w1 = false, w2 = false;
  int z0 = -1, z1 = -1, z2 = -1;
  const bool f0 = active && (idx[0] == 0 || idx[0] == K);
  const bool f1 = active && (idx[1] == 0 || idx[1] == K);
  const bool f2 = (D == 3) && active && (idx[2] == 0 || idx[2] == K);
  if (f0) gather_nb<R, K, D, RAIN, 0>(item, ec, e, n, idx[0], U, auxT, auxS, N, nb0, w0, z0);
  if (f1) gather_nb<R, K, D, RAIN, 1>(item, ec, e, n, idx[1], U, auxT, auxS, N, nb1, w1, z1);
  if constexpr (D == 3) {
    if (f2) gather_nb<R, K, D, RAIN, 2>(item, ec, e, n, idx[2], U, auxT, auxS, N, nb2, w2, z2);
  }
  Pt<R, D, RAIN> q;
  eval_point<R, D, RAIN>(a, Uq, T, rvs, active ? iz : item.hoff, q);
  R Rv[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) Rv[v] = R(0);
  stage_flux<R, K, D, RAIN, 0>(q, sF[0]);
  stage_flux<R, K, D, RAIN, 1>(q, sF[1]);
  if constexpr (D == 3) stage_flux<R, K, D, RAIN, 2>(q, sF[2]);
  __syncthreads();
  if (active) {
    volume_dir<R, K, D, RAIN, 0>(md, idx[0], sF[0], Rv, sD);
    volume_dir<R, K, D, RAIN, 1>(md, idx[1], sF[1], Rv, sD);
    if constexpr (D == 3) volume_dir<R, K, D, RAIN, 2>(md, idx[2], sF[2], Rv, sD);
  }
  if (f0) face_dir<R, K, D, RAIN, 0>(a, item, md, idx[0], iz, Uq, q, nb0, w0, z0, Rv);
  if (f1) face_dir<R, K, D, RAIN, 1>(a, item, md, idx[1], iz, Uq, q, nb1, w1, z1, Rv);
  if constexpr (D == 3) {
    if (f2) face_dir<R, K, D, RAIN, 2>(a, item, md, idx[2], iz, Uq, q, nb2, w2, z2, Rv);
  }
  int iters = 0, bad = 0;
  if (active) {
    sources<R, D, RAIN>(a, Uq, q, Rv);
    if (flags & kSip) {
#pragma unroll
      for (int v = 0; v < NV; ++v) Rv[v] += (((const R*)a.sip_out) + (size_t)v * N)[g];
    }
    if (MODE == 0) {
#pragma unroll
      for (int v = 0; v < NV; ++v) (out + (size_t)v * N)[g] = Rv[v];
    } else {
      const R k2 = (R)(c2 * (dt_m ? dt_m[item.member] : 1.0));
      const R k1 = (R)c1;
      R Un[NV];
      if (c0 != 0.0) {
        const R k0 = (R)c0;
#pragma unroll
        for (int v = 0; v < NV; ++v) Un[v] = k0 * (U0 + (size_t)v * N)[g] + k1 * Uq[v] + k2 * Rv[v];
      } else {
#pragma unroll
        for (int v = 0; v < NV; ++v) Un[v] = k1 * Uq[v] + k2 * Rv[v];
      }
      if (MODE != 0 && (flags & kSponge)) sponge_point<R, D, RAIN>(a, iz, Un);
#pragma unroll
      for (int v = 0; v < NV; ++v) (out + (size_t)v * N)[g] = Un[v];
      if (MODE == 2) {
        // split of the new state (FP64), warm-started at this node's (T, rho_vs)
        const Bg bg = bg_at(a, iz);
        const double rd = bg.rd + (double)Un[V::RD];
        const double rm = bg.rm + (double)Un[V::RM];
        const double rr = RAIN ? bg.rr + (double)Un[V::RR] : 0.0;
        double ke = 0.0;
#pragma unroll
        for (int i = 0; i < D; ++i) {
          const double mi = (double)Un[V::M0 + i];
          ke += mi * mi;
        }
        const double re = bg.E + (double)Un[V::E] - 0.5 * ke * rcp64(rd + rm + rr);
        const SplitOut s = split_warm<D>(a, rd, rm, rr, re, T, rvs);
        iters = s.iters;
        bad = s.bad;
        oT[g] = s.T;
        oS[g] = ((flags & kRefreshRvs) && s.bad == 0) ? rho_vs(a, s.T) : s.rvs;
      }
    }
  }
  if (MODE == 2) record_stats(a, seen, iters, bad);
}

// one work item per block
// FP32 in 2D (Q2 and up): 7 wavefronts per SIMD, what the LDS allows; with rain it
// allows 6 at Q3, Q4, Q5 and Q7 (a bound above that would be none).  Left at 5
// (94 registers, which only the split's rarely taken slow path needs) the kernel
// waits for memory half of its time; bound to 72 or 80 registers that path spills a
// few values and the rest does not.  64 members of 160 x 80 Q3 at most, five steps:
// 2.83 ms at 5, 2.75 at 6, 2.61 at 7.  About 980 000 nodes, two steps, left at 5
// against bound: Q2 324 -> 273 us, Q3 214 -> 202, Q4 236 -> 219, Q5 224 -> 209, Q6
// 242 -> 217, Q7 220 -> 205; with rain Q2 357 -> 301, Q3 238 -> 224, Q4 254 -> 245,
// Q5 242 -> 236, Q6 256 -> 243, Q7 236 -> 226.  Q1 takes another path, which spills in
// its loops at 6 (390 -> 545 us).  In 3D the LDS holds it at 5.  FP64 kernels are left
// to the compiler: 2D Q2 to Q7 measured the same at 5 and 6.
template <typename R, int K, int D, int RAIN>
constexpr int min_waves() {
  if (sizeof(R) == 8) return 1;
  return D == 2 && K >= 2 ? (RAIN && K != 2 && K != 6 ? 6 : 7) : 4;
}

template <typename R, int K, int D, int RAIN, int MODE>
__global__ void __launch_bounds__(block_kernel_threads(K, D, 256)) __attribute__((amdgpu_waves_per_eu(min_waves<R, K, D, RAIN>())))
rhs_kernel(KArgs a, const R* __restrict__ U, const double* __restrict__ auxT,
           const double* __restrict__ auxS, R* __restrict__ out, const R* __restrict__ U0,
           const double* __restrict__ dt_m, double c0, double c1, double c2,
           double* __restrict__ oT, double* __restrict__ oS, int flags) {
  using S = Shape<K, D, block_threads<R>()>;
  using V = Vars<D, RAIN>;
  constexpr int P1 = S::P1;
  constexpr bool PAIRS = K >= 2;
  __shared__ R sF[D][V::NV * S::NT];
  __shared__ R sD[P1 * P1];
  __shared__ R sU[PAIRS ? V::NV * S::NT : 1];
  __shared__ R sL[PAIRS ? D * S::NT : 1];
  __shared__ ElemTab<D> tab[PAIRS && D == 3 ? S::EPB : 1];
  __shared__ R sC[PAIRS && D == 2 && Lds2d<R, K, RAIN>::SEP ? V::NV * Lds2d<R, K, RAIN>::NQ : 1];
  if (threadIdx.x < P1 * P1) sD[threadIdx.x] = (R)a.Dhat[threadIdx.x];
  const ItemWalk walk(a.nitems, a.walk_rev);
  const int it_ = walk.item(0);
  if (it_ < 0) return;
  if constexpr (PAIRS && D == 3)
    rhs_item_3d<R, K, RAIN, MODE>(a, threadIdx.x, it_, tab, &sF[0][0], sU, sL, sD, U, auxT, auxS, out, U0, dt_m, c0,
                                  c1, c2, oT, oS, flags);
  else if constexpr (PAIRS) {
    __syncthreads();   // sD
    rhs_item_2d<R, K, RAIN, MODE>(a, threadIdx.x, it_, &sF[0][0], sU, sL, sC, sD, U, auxT, auxS, out, U0, dt_m, c0,
                                  c1, c2, oT, oS, flags);
  }
  else
    rhs_item<R, K, D, RAIN, MODE>(a, threadIdx.x, it_, sF, sD, U, auxT, auxS, out, U0, dt_m, c0, c1, c2, oT, oS, flags);
}

// FP32: 4 wavefronts per SIMD, four blocks per CU; at 2D Q2, whose blocks have 6
// wavefronts, 5 (470 x 230, 4 blocks per CU, two steps: 468 us at 4, where two
// blocks fit, 372 at 5; 6 spills in the loop).  At Q1 the loop used to
// keep the argument block's values in registers: 189 spilled at 3D Q1, 22 now,
// 64 x 60 x 30, 4 blocks per CU 958 -> 355 us.
template <typename R, int K, int D>
constexpr int persistent_waves() { return sizeof(R) == 4 ? (block_kernel_threads(K, D, 256) > 256 ? 5 : 4) : 1; }

// persistent: a grid smaller than the item count walks the items
template <typename R, int K, int D, int RAIN, int MODE>
__global__ void __launch_bounds__(block_kernel_threads(K, D, 256)) __attribute__((amdgpu_waves_per_eu(persistent_waves<R, K, D>())))
rhs_kernel_persistent(KArgs a, const KArgs* __restrict__ a_dev, const R* __restrict__ U,
                      const double* __restrict__ auxT,
                      const double* __restrict__ auxS, R* __restrict__ out, const R* __restrict__ U0,
                      const double* __restrict__ dt_m, double c0, double c1, double c2,
                      double* __restrict__ oT, double* __restrict__ oS, int flags) {
  using S = Shape<K, D, block_threads<R>()>;
  using V = Vars<D, RAIN>;
  constexpr int P1 = S::P1;
  constexpr bool PAIRS = K >= 2;
  __shared__ R sF[D][V::NV * S::NT];
  __shared__ R sD[P1 * P1];
  __shared__ R sU[PAIRS ? V::NV * S::NT : 1];
  __shared__ R sL[PAIRS ? D * S::NT : 1];
  __shared__ ElemTab<D> tab[PAIRS && D == 3 ? S::EPB : 1];
  __shared__ R sC[PAIRS && D == 2 && Lds2d<R, K, RAIN>::SEP ? V::NV * Lds2d<R, K, RAIN>::NQ : 1];
  if (threadIdx.x < P1 * P1) sD[threadIdx.x] = (R)a.Dhat[threadIdx.x];
  const ItemWalk walk(a.nitems);
#pragma clang loop unroll(disable)
  for (int kk = 0;; ++kk) {
    const int it_ = walk.item(kk);
    if (it_ < 0) break;
    // The argument block (its device copy a_dev) and the thread index pass
    // through opaque copies in every iteration: constants and per-thread
    // values hoisted out of the loop would stay live across it and exhaust
    // the registers.
    unsigned long long apv = (unsigned long long)a_dev;
    asm volatile("" : "+s"(apv));
    // constant address space: the block is read-only during the launch, so
    // its fields are scalar loads
    const KArgs DGM_AS_CONST* ap = (const KArgs DGM_AS_CONST*)apv;
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    if constexpr (PAIRS && D == 3)
      rhs_item_3d<R, K, RAIN, MODE>(*ap, t, it_, tab, &sF[0][0], sU, sL, sD, U, auxT, auxS, out, U0, dt_m, c0, c1, c2,
                                    oT, oS, flags);
    else if constexpr (PAIRS)
      rhs_item_2d<R, K, RAIN, MODE>(*ap, t, it_, &sF[0][0], sU, sL, sC, sD, U, auxT, auxS, out, U0, dt_m, c0, c1, c2,
                                    oT, oS, flags);
    else if constexpr (sizeof(R) == 4)
      rhs_item<R, K, D, RAIN, MODE>(*ap, t, it_, sF, sD, U, auxT, auxS, out, U0, dt_m, c0, c1, c2, oT, oS, flags);
    else
      // (FP64 has the registers; through ap it rounds differently from rhs_kernel)
      rhs_item<R, K, D, RAIN, MODE>(a, threadIdx.x, it_, sF, sD, U, auxT, auxS, out, U0, dt_m, c0, c1, c2, oT, oS, flags);
    __syncthreads();   // the LDS tiles are reused by the next item
  }
}



// ---------------------------------------------------------------------------
// conservation diagnostics: per-block FP64 partial sums in a fixed order
// ---------------------------------------------------------------------------
template <typename R, int K, int D, int RAIN>
__global__ void __launch_bounds__(256)
mass_kernel(KArgs a, int item0, const R* __restrict__ U, double* __restrict__ partial) {
  // (blocks map to items in order here: partials are summed in a fixed order)
  using S = Shape<K, D, block_threads<R>()>;
  using V = Vars<D, RAIN>;
  constexpr int P1 = S::P1, NP = S::NP;
  __shared__ double sm[3][S::NT];
  const int NT = blockDim.x;
  const int t = threadIdx.x;
  const Item item = a.items[item0 + blockIdx.x];
  const MemberDesc& md = a.mem[item.member];
  const int le = t / NP, n = t - le * NP;
  const int e = item.e0 + le;
  double md_ = 0.0, mw = 0.0, fl = 0.0;
  if (e < item.ne) {
    const size_t N = a.nnodes;
    const size_t g = (size_t)(item.eoff + e) * NP + n;
    int idx[3] = {n % P1, (n / P1) % P1, (D == 3) ? n / (P1 * P1) : 0};
    double w = md.J;
#pragma unroll
    for (int j = 0; j < D; ++j) w *= a.w[idx[j]];
    md_ = w * (double)U[V::RD * N + g];
    mw = w * ((double)U[V::RM * N + g] + (RAIN ? (double)U[V::RR * N + g] : 0.0));
    // rain through the slip walls: with Lobatto nodes the wall is a node
    // layer; with Gauss nodes the thread of the lowest (highest) node of each
    // vertical line takes the trace of rho_r' along it at the floor (lid),
    // plus the background's face trace
    if (RAIN && item.bc[D - 1] == 1) {
      const ElemCoord<D> ec = item_coord<D>(item, le);
      const int l = idx[D - 1];
      const bool bottom = ec.c[D - 1] == 0 && l == 0;
      const bool top = ec.c[D - 1] == item.n[D - 1] - 1 && l == K;
      if (bottom || top) {
        double rr;
        if (a.basis == 0) {
          rr = a.bg_rr[item.hoff + ec.c[D - 1] * P1 + l] + (double)U[V::RR * N + g];
        } else {
          constexpr int ZS = (D == 2) ? P1 : P1 * P1;   // node stride along the vertical
          const double* Lt = bottom ? a.gl_m : a.gl_p;
          const size_t g0 = g - (size_t)l * ZS;
          double tr = 0.0;
          for (int m = 0; m < P1; ++m) tr += Lt[m] * (double)U[V::RR * N + g0 + (size_t)m * ZS];
          const int row = item.hoff / P1 + ec.c[D - 1];
          rr = a.bgf[2 * a.bgf_n + 2 * row + (bottom ? 0 : 1)] + tr;
        }
        double vr = a.vr_const;
        if (a.vr_mode != 0) vr = rr > 0.0 ? a.vr_pref * pow(rr, 0.125) : 0.0;
        double wf = md.face_J[D - 1];
#pragma unroll
        for (int j = 0; j < D - 1; ++j) wf *= a.w[idx[j]];
        // wall flux of rain is -rho_r v_r along +e_z: out at the floor, in at the lid
        fl = bottom ? wf * rr * vr : -wf * rr * vr;
      }
    }
  }
  sm[0][t] = md_; sm[1][t] = mw; sm[2][t] = fl;
  __syncthreads();
  // fixed-order tree over the block (NT need not be a power of two)
  for (int s = 1; s < NT; s <<= 1) {
    if ((t % (2 * s)) == 0 && t + s < NT) {
      sm[0][t] += sm[0][t + s];
      sm[1][t] += sm[1][t + s];
      sm[2][t] += sm[2][t + s];
    }
    __syncthreads();
  }
  if (t == 0) {
    partial[3 * blockIdx.x + 0] = sm[0][0];
    partial[3 * blockIdx.x + 1] = sm[1][0];
    partial[3 * blockIdx.x + 2] = sm[2][0];
  }
}

// ---------------------------------------------------------------------------
// transpose of the end-of-step sponge (the adjoint of dg_rk_step)
// ---------------------------------------------------------------------------
// Wp = S^T W for the pointwise sponge map S of sponge_point:
//   Wp[rho_d] = W[rho_d],  Wp[rho_m] = (1 - delta) W[rho_m] + delta W[rho_d],
//   Wp[rho_r] = (1 - delta) W[rho_r] + delta W[rho_d],  Wp[v] = (1 - delta) W[v]
//   for the momentum and E'.
template <typename R, int K, int D, int RAIN>
__global__ void __launch_bounds__(256)
sponge_vjp_kernel(KArgs a, const R* __restrict__ W, R* __restrict__ Wp) {
  using S = Shape<K, D, block_threads<R>()>;
  using V = Vars<D, RAIN>;
  constexpr int P1 = S::P1, NP = S::NP, NV = V::NV;
  const ItemWalk walk(a.nitems);
  for (int k = 0;; ++k) {
    const int it_ = walk.item(k);
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
    const R dl = (R)a.sponge[item.hoff + ec.c[D - 1] * P1 + l];
    const R keep = R(1) - dl;
    const R wd = ld(W, N, V::RD, g);
    st(Wp, N, V::RD, g, wd);
    st(Wp, N, V::RM, g, keep * ld(W, N, V::RM, g) + dl * wd);
    if (RAIN) st(Wp, N, V::RR, g, keep * ld(W, N, V::RR, g) + dl * wd);
#pragma unroll
    for (int v = V::M0; v < NV; ++v) st(Wp, N, v, g, keep * ld(W, N, v, g));
  }
}

}  // namespace dgm
