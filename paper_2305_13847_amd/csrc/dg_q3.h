// Stage kernel for Q3 hexahedra (Lobatto basis): one wavefront per element, a
// 2 x 2 brick (x, y) of elements per block (Brick; thinner on columns and slabs).
//
// A Q3 hexahedron has (3+1)^3 = 64 nodes, so lane n of a wavefront owns node
// n = i + 4 j + 16 l of one element.  Everything that depends on the element
// alone (its coordinates, neighbours, wall flags, offsets) is wave-uniform and
// lives in scalar registers; per-lane indices are bit fields of the lane id.
// Each wavefront works in its own LDS tiles; the block meets once, after the
// fluxes are staged (with diffusion twice more, for the viscous ones), so that the
// faces inside the brick take both sides from LDS.  With partners on one x and one y side an element has four outer
// faces, 64 face nodes: one full pass of its lanes evaluates the neighbours
// (a single row of elements has 96, two passes with one half empty).
//
// Per element and RK stage (Section 3.2 weak form, Section 3.3 mass and
// update, Section 3.4 split):
//   1. load U, (T, rho_vs) of every node, and the background at the
//      element's heights and the neighbours' face heights into a small LDS
//      table; issue the loads of the outer faces' neighbour traces at once
//      (their addresses depend on the element only);
//   2. evaluate the point state (FP64 reconstruction of p' and rho e), stage
//      F_x, F_y, F_z and, for the partners, U and the wave speeds at the faces
//      inside the brick in LDS; the sources;
//   3. volume term from the LDS lines;
//   4. faces: each lane evaluates one outer neighbour trace (on a slip wall
//      its own, mirrored), forms the Lax-Friedrichs flux with the own trace
//      (state across the lanes, flux from LDS), and leaves the lifted
//      correction in LDS; the faces inside
//      the brick need no evaluation;
//   5. every node adds the corrections of its faces, then the stage update,
//      the sponge, the store and the split of the new state (stage_epilogue).
//
// Bound by HBM traffic and VALU issue together: on 64 x 64 x 32 in FP32 a stage
// takes 255 us and moves 1.04 GB (0.66 GB is algorithmic, the rest neighbour data
// that the L2s miss), 86 % of a copy's rate, with the VALU 76 % busy.  Five steps
// 5.73 -> 5.20 ms against one element per wavefront without bricks (four blocks per
// CU, 30 % more L2 requests).  FP64, 33 x 31 x 17, two steps: 580 us without bricks,
// 545 with 2 x 1 bricks and a tile of the state, 485 now; 64 x 64 x 32 4.25 -> 3.84.
#pragma once
#include "dg_kernels.h"

namespace dgm {

// Order LDS traffic of one wavefront: its earlier LDS writes are visible to
// its later reads (LDS operations of a wavefront complete in order; the fences
// keep the compiler from moving memory operations across).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Volume term from this wavefront's flux tiles (rows of 64 nodes), variable
// by variable: R_v += sum_J (2/h_J) sum_b Dhat[i_J][b] F_J,v(node b on the
// lane's J-line).  The scheduling barrier after each variable keeps the
// compiler from issuing all 84 LDS reads at once (their results would need
// more registers than the kernel has).
template <typename R, int RAIN>
__device__ __forceinline__ void volume_q3(const MemberDesc& md, int li, int lj, int ll, int lane,
                                          const R (*sF)[Vars<3, RAIN>::NV][64], R* Rv, const R* sD) {
  constexpr int NV = Vars<3, RAIN>::NV;
  const R sx = (R)md.two_over_h[0], sy = (R)md.two_over_h[1], sz = (R)md.two_over_h[2];
  const int bx = lane - li, by = lane - 4 * lj, bz = lane - 16 * ll;
  R dx[4], dy[4], dz[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    dx[b] = sD[li * 4 + b];
    dy[b] = sD[lj * 4 + b];
    dz[b] = sD[ll * 4 + b];
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    R ax = dx[0] * sF[0][v][bx], ay = dy[0] * sF[1][v][by], az = dz[0] * sF[2][v][bz];
#pragma unroll
    for (int b = 1; b < 4; ++b) {
      ax += dx[b] * sF[0][v][bx + b];
      ay += dy[b] * sF[1][v][by + 4 * b];
      az += dz[b] * sF[2][v][bz + 16 * b];
    }
    Rv[v] += sx * ax;
    Rv[v] += sy * ay;
    Rv[v] += sz * az;
    // (keep the sums here: sunk to their use behind the faces, every LDS value
    // would stay in registers until then)
    asm volatile("" : "+v"(Rv[v]));
    __builtin_amdgcn_sched_barrier(0);
  }
}

// background of one height from a wavefront's LDS table
__device__ __forceinline__ Bg q3_bg(const double2* b) {
  const double2 x = b[0], y = b[1], z = b[2];
  return Bg{x.x, x.y, y.x, y.y, z.x, z.y};
}

// A face task: a face node of this element and the neighbour's matching node.
struct FaceTask {
  int n, J, side, h;   // own node, direction, side, row of the background table
  bool wall;
  unsigned gn;         // global node to read (on a wall the own one, mirrored)
};

// Task of face node (ta, tb) on side `side` of direction J: `de` is the step to
// the neighbour's element, gbase the element's first node.
__device__ __forceinline__ FaceTask face_task(int J, int side, int ta, int tb, bool wall, int de, unsigned gbase) {
  constexpr int K = 3;
  FaceTask f;
  f.J = J;
  f.side = side;
  f.wall = wall;
  int match;
  f.n = face_node<K, 3>(J, side, ta, tb, match);
  f.gn = gbase + (unsigned)(f.n + (wall ? 0 : de * 64 + match));
  f.h = J == 2 ? (wall ? (side ? K : 0) : (side ? 5 : 4)) : tb;
  return f;
}

// Outer face task: evaluate the neighbour's trace, the Lax-Friedrichs flux with
// the own trace (Uo; its wave speed along z, lz; the others in LDS); the
// correction replaces F_J at the own node.
template <typename R, int RAIN>
__device__ __forceinline__ void q3_outer(const KArgs& a, const FaceTask& f, Pair<R, 3, RAIN>& nb,
                                         R (*sF)[Vars<3, RAIN>::NV][64], const R* Uo, R lz, const R (*sL)[32],
                                         const double2 (*sB)[kBgStride / 2], R hx, R hy, R hz) {
  using V = Vars<3, RAIN>;
  constexpr int NV = V::NV;
  const int J = f.J;
#pragma unroll
  for (int i = 0; i < 3; ++i) nb.nb.U[V::M0 + i] = f.wall && i == J ? -nb.nb.U[V::M0 + i] : nb.nb.U[V::M0 + i];
  Pt<R, 3, RAIN> qn;
  eval_bg<R, 3, RAIN>(a, nb.nb.U, nb.nb.T, nb.nb.rvs, q3_bg(sB[f.h]), qn);
  const R uj = J == 0 ? qn.u[0] : (J == 1 ? qn.u[1] : qn.u[2]);
  R Fn[NV];
  flux_sel<R, 3, RAIN>(qn, J, uj, Fn);
  R ln = fabs(uj) + qn.cm;
  if (RAIN) ln += J == 2 ? fabs(qn.vr) : R(0);
  const R lo = J == 2 ? lz : sL[J & 1][f.side * 16 + (int)(threadIdx.x & 15)];
  // Lambda = max over the two sides, ties to the minus side
  const bool own = f.side ? (lo >= ln) : !(ln >= lo);
  const R hl = J == 0 ? hx : (J == 1 ? hy : hz);
  const R kf = f.side ? -hl : hl;
  const R kj = hl * (own ? lo : ln);
#pragma unroll
  for (int v = 0; v < NV; ++v) sF[J][v][f.n] = fma(kf, sF[J][v][f.n] + Fn[v], kj * (nb.nb.U[v] - Uo[v]));
}

__device__ __forceinline__ bool q3_wall(int bc, int c, int n, int side) { return bc == 1 && (side ? c == n - 1 : c == 0); }
// step to the neighbour's coordinate (periodic wrap)
__device__ __forceinline__ int q3_step(int c, int n, int side) {
  return side ? (c == n - 1 ? 1 - n : 1) : (c == 0 ? n - 1 : -1);
}

// ---------------------------------------------------------------------------
// Artificial diffusion (Section 3.5, the form in dg_sip.h) inside the stage
// kernel: the tendency starts from S = -M^{-1} A_h instead of zero, in the tiles
// that the fluxes use afterwards.
//   1. the vertex means of alpha_K (27 elements share this one's vertices) and
//      the Q1 viscosity at the nodes;
//   2. the viscous fluxes -alpha G_j to LDS, their volume term;
//   3. at each face point alpha [U] and alpha ({G_j} - tau [U]): the outer faces'
//      neighbour gradients from their lines in memory, the inner ones' from the
//      partner's tile;
//   4. both lifted to the nodes of the point's line.
// A separate kernel wrote the tendency and the stage kernel read it (165 MB and
// 35 us a stage at 48 x 40 x 24 in FP32), loaded the state and its neighbours a
// second time, and took the vertex means from a third kernel.  48 x 40 x 24 with
// rain, two SSPRK(4,3) steps: FP32 1.82 -> 1.53 ms, FP64 3.9 -> 3.1; 5 x 4 x 3
// (launches) 0.2 -> 0.12.  Bound by VALU issue (70 % busy, 1690 instructions per
// element against 800 without diffusion) at 4 wavefronts per SIMD.
// ---------------------------------------------------------------------------

// The neighbour's line behind an outer face point, from the face inwards.
template <typename R, int RAIN>
struct SipLine {
  R u[4][Vars<3, RAIN>::NV];
};

template <typename R, int RAIN>
__device__ __forceinline__ void sip_line_load(const R* __restrict__ U, unsigned N, const FaceTask& f,
                                              SipLine<R, RAIN>& l) {
  const int str = f.J == 0 ? 1 : (f.J == 1 ? 4 : 16);
  // (on a wall gn is the own node: inwards is the other way; the values are not used)
  const int step = (f.side != 0) != f.wall ? str : -str;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
#pragma unroll
    for (int v = 0; v < Vars<3, RAIN>::NV; ++v) l.u[b][v] = ld(U, N, v, f.gn + (unsigned)(b * step));
  }
}

// alpha [U] and alpha ({G_J} - tau_J [U]) at a face point, [U] lower minus upper
// (a0, a1: the viscosities there).
template <typename R, int RAIN>
struct SipPoint {
  R j[Vars<3, RAIN>::NV], q[Vars<3, RAIN>::NV];
};

template <typename R, int RAIN>
__device__ __forceinline__ void sip_outer(const MemberDesc& md, const FaceTask& f, const SipLine<R, RAIN>& l,
                                          const R* Dm, const R (*sF)[Vars<3, RAIN>::NV][64], const R (*sU)[64],
                                          R a0, R a1, SipPoint<R, RAIN>& p) {
  using V = Vars<3, RAIN>;
  const int J = f.J;
  const R dj = (R)(J == 0 ? md.two_over_h[0] : (J == 1 ? md.two_over_h[1] : md.two_over_h[2]));
  const R ct = (R)(J == 0 ? md.sip_tau[0] : (J == 1 ? md.sip_tau[1] : md.sip_tau[2]));
  // the end rows of D are each other's negative mirror image
  const R sg = f.side ? dj : -dj;
  R w[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) w[b] = sg * Dm[b];
#pragma unroll
  for (int v = 0; v < V::NV; ++v) {
    const R al = RAIN && v == V::RR ? a1 : a0;
    R gn = w[0] * l.u[0][v];
#pragma unroll
    for (int b = 1; b < 4; ++b) gn = fma(w[b], l.u[b][v], gn);
    const R uo = sU[v][f.n], d = uo - l.u[0][v];
    const R ju = al * (f.side ? d : -d);
    const R q = R(0.5) * (al * gn - sF[J][v][f.n]) - ct * ju;
    p.j[v] = f.wall ? R(0) : ju;
    p.q[v] = f.wall ? R(0) : q;
  }
}

// The viscosity of both fields at this lane's node.  sK: scratch of 70 doubles.
template <typename R, int RAIN>
__device__ __forceinline__ void sip_viscosity(const KArgs& a, const Item& item, int ex, int ey, int ez, int lane, int li,
                                              int lj, int ll, double k0, double k1, double* sK, R& al0, R& al1) {
  if (lane < 27) {
    sK[lane] = k0;
    if (RAIN) sK[27 + lane] = k1;
  }
  wave_lds_sync();
  if (lane < (RAIN ? 16 : 8)) {
    const int cx = lane & 1, cy = (lane >> 1) & 1, cz = (lane >> 2) & 1;
    const double* k = sK + (lane >> 3) * 27 + 13 + cx + 3 * cy + 9 * cz;
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < 8; ++c) s += k[-((c & 1) + 3 * ((c >> 1) & 1) + 9 * (c >> 2))];
    // a vertex on a wall is shared by half as many elements (their entries are 0)
    const bool wx = item.bc[0] == 1 && ex == (cx ? item.n[0] - 1 : 0);
    const bool wy = item.bc[1] == 1 && ey == (cy ? item.n[1] - 1 : 0);
    const bool wz = item.bc[2] == 1 && ez == (cz ? item.n[2] - 1 : 0);
    s *= 0.125 * (wx ? 2.0 : 1.0) * (wy ? 2.0 : 1.0) * (wz ? 2.0 : 1.0);
    sK[54 + lane] = s;
  }
  wave_lds_sync();
  const double p1 = 0.5 * (1.0 + a.xn[1]), p2 = 0.5 * (1.0 + a.xn[2]);
  auto up = [&](int i) { return i == 0 ? 0.0 : (i == 1 ? p1 : (i == 2 ? p2 : 1.0)); };
  const double px = up(li), py = up(lj), pz = up(ll);
  auto at = [&](const double* v) {
    double r[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const double y0 = (1.0 - px) * v[4 * c] + px * v[4 * c + 1];
      const double y1 = (1.0 - px) * v[4 * c + 2] + px * v[4 * c + 3];
      r[c] = (1.0 - py) * y0 + py * y1;
    }
    return (R)((1.0 - pz) * r[0] + pz * r[1]);
  };
  al0 = at(sK + 54);
  al1 = RAIN ? at(sK + 62) : al0;
  wave_lds_sync();
}

// FP32: 5 wavefronts per SIMD, 96 registers (six fit the LDS, but the split's
// slow path then spills and the blocks in flight outgrow the L2s: 64 x 64 x 32,
// five steps, 5.15 -> 5.35 ms).  FP64: 3, what the LDS allows.  With diffusion
// the tile of the state and its registers leave 4 and 2.
template <typename R, int SIP>
constexpr int q3_min_waves() { return sizeof(R) == 4 ? (SIP ? 4 : 5) : (SIP ? 2 : 3); }

template <typename R, int RAIN, int MODE, int SIP, int BX, int BY>
__global__ void __launch_bounds__(64 * BX * BY)
__attribute__((amdgpu_waves_per_eu(q3_min_waves<R, SIP>())))
rhs_q3_kernel(KArgs a, const R* __restrict__ U, const double* __restrict__ auxT,
              const double* __restrict__ auxS, R* __restrict__ out, const R* __restrict__ U0,
              const double* __restrict__ dt_m, double c0, double c1, double c2, double* __restrict__ oT,
              double* __restrict__ oS, int flags) {
  constexpr int K = 3, P1 = 4, NP = 64, D = 3;
  using V = Vars<D, RAIN>;
  constexpr int NV = V::NV;
  constexpr int WPB = BX * BY;   // wavefronts (elements) per block
  // per-wavefront LDS tiles: fluxes of the three directions (later the face
  // corrections), and what the faces inside the brick need of the state and the
  // wave speeds
  __shared__ alignas(16) R sF_all[WPB][D][NV][NP];   // (diffusion: also doubles)
  __shared__ R sI_all[SIP ? 1 : WPB][2][NV][P1 * P1];   // state at the nodes of the inner x and y face
  __shared__ R sL_all[WPB][2][2 * P1 * P1];   // along x and y at the face nodes: side, face node
  __shared__ R sU_all[SIP ? WPB : 1][NV][SIP ? NP : 1];   // (with diffusion, whose gradients need it) all of it
  // background (KArgs::bgt fields) at the brick's four heights and at the face
  // heights of the neighbours below and above: the same for its elements, and
  // each wavefront writes all of it (the same values) before it reads
  __shared__ double2 sB[6][kBgStride / 2];
  __shared__ R sD[P1 * P1], sDm[SIP ? P1 * P1 : 1];
  if (!SIP && threadIdx.x < P1 * P1) sD[threadIdx.x] = (R)a.Dhat[threadIdx.x];

  const ItemWalk walk(a.nbricks, a.walk_rev);
  const int it_ = walk.item(0);
  if (it_ < 0) return;                     // block-uniform
  const int seen = MODE == 2 ? stats_seen(a) : 0;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = (int)(threadIdx.x & 63);
  const Item item = a.bricks[it_];
  const MemberDesc& md = a.mem[item.member];
  R(*sF)[NV][NP] = sF_all[w];
  R(*sI)[NV][P1 * P1] = sI_all[SIP ? 0 : w];
  R(*sL)[2 * P1 * P1] = sL_all[w];

  // element (scalar): coordinates, partners inside the brick, outer faces
  const int n0 = item.n[0], n1 = item.n[1], n2 = item.n[2];
  const int b0 = item.bc[0], b1 = item.bc[1], b2 = item.bc[2];
  const Brick<BX, BY> br(item, w);
  const int dx = br.dx, dy = br.dy, ex = br.ex, ey = br.ey, ez = br.ez;
  const bool act = br.act, px = br.px, py = br.py;   // wave-uniform
  const int e = item.e0 + dx + dy * n0;
  const unsigned N = a.nnodes;
  const unsigned gbase = (unsigned)(item.eoff + e) * NP;   // first node of the element
  const unsigned g = gbase + lane;
  const int li = lane & 3, lj = (lane >> 2) & 3, ll = lane >> 4;
  const int izb = item.hoff + ez * P1;                     // first height index of the element
  const int iz = izb + ll;

  // outer face tasks, 16 lanes per face: x and y on the side away from the
  // brick, z below and above
  const int tf = lane >> 4, ta = lane & 3, tb = (lane >> 2) & 3;
  const bool wx = q3_wall(b0, ex, n0, dx), wy = q3_wall(b1, ey, n1, dy);
  const bool wz0 = q3_wall(b2, ez, n2, 0), wz1 = q3_wall(b2, ez, n2, 1);
  const int nn01 = n0 * n1;
  const int qx = q3_step(ex, n0, dx), qy = q3_step(ey, n1, dy) * n0;
  const int qz0 = q3_step(ez, n2, 0) * nn01, qz1 = q3_step(ez, n2, 1) * nn01;
  const FaceTask f0 = face_task(tf < 2 ? tf : 2, tf == 0 ? dx : (tf == 1 ? dy : tf - 2), ta, tb,
                                tf == 0 ? wx : (tf == 1 ? wy : (tf == 2 ? wz0 : wz1)),
                                tf == 0 ? qx : (tf == 1 ? qy : (tf == 2 ? qz0 : qz1)), gbase);
  // and, without a partner, the far sides: lanes 0..15 x, 16..31 y
  const FaceTask f1 = face_task(tf & 1, 1, ta, tb, (tf & 1) ? q3_wall(b1, ey, n1, 1) : q3_wall(b0, ex, n0, 1),
                                (tf & 1) ? q3_step(ey, n1, 1) * n0 : q3_step(ex, n0, 1), gbase);
  const bool far1 = (tf == 0 && !px) || (tf == 1 && !py);

  R Uq[NV], Rv[NV];
  double T = 300.0, rvs = 0.0;
  R lz = R(0);
  Pair<R, D, RAIN> nb0;
#pragma unroll
  for (int v = 0; v < NV; ++v) Rv[v] = R(0);
  if constexpr (SIP) {
    R(*sU)[NP] = sU_all[w];
    R al0 = R(0), al1 = R(0);
    R Dm[P1];
#pragma unroll
    for (int b = 0; b < P1; ++b) Dm[b] = (R)a.Dm[b];
    SipLine<R, RAIN> l0;
    if (act) {
      // alpha_K of the elements around this one (0 beyond a wall)
      double k0 = 0.0, k1 = 0.0;
      if (lane < 27) {
        const int oz = lane / 9, oy = (lane - 9 * oz) / 3, ox = lane - 9 * oz - 3 * oy;
        int cx = ex + ox - 1, cy = ey + oy - 1, cz = ez + oz - 1;
        const bool in = (b0 == 0 || (cx >= 0 && cx < n0)) && (b1 == 0 || (cy >= 0 && cy < n1)) &&
                        (b2 == 0 || (cz >= 0 && cz < n2));
        cx = cx < 0 ? cx + n0 : (cx >= n0 ? cx - n0 : cx);
        cy = cy < 0 ? cy + n1 : (cy >= n1 ? cy - n1 : cy);
        cz = cz < 0 ? cz + n2 : (cz >= n2 ? cz - n2 : cz);
        if (in) {
          const unsigned ek = (unsigned)(item.eoff + cx + n0 * (cy + n1 * cz));
          k0 = a.sip_aK[ek];
          if (RAIN) k1 = a.sip_aK[a.etot + ek];
        }
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) Uq[v] = ld(U, N, v, g);
      sip_line_load<R, RAIN>(U, N, f0, l0);
      const R dh = lane < P1 * P1 ? (R)a.Dhat[lane] : R(0), dm = lane < P1 * P1 ? (R)a.Dm[lane] : R(0);
      // (every wavefront writes the same tables before it reads)
      if (lane < P1 * P1) {
        sD[lane] = dh;
        sDm[lane] = dm;
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) sU[v][lane] = Uq[v];
      sip_viscosity<R, RAIN>(a, item, ex, ey, ez, lane, li, lj, ll, k0, k1, (double*)&sF[0][0][0], al0, al1);
      const R d0 = (R)md.two_over_h[0], d1 = (R)md.two_over_h[1], d2 = (R)md.two_over_h[2];
      const int bx = lane - li, by = lane - P1 * lj, bz = lane - 16 * ll;
      R wx_[P1], wy_[P1], wz_[P1];
#pragma unroll
      for (int b = 0; b < P1; ++b) {
        wx_[b] = d0 * sDm[li * P1 + b];
        wy_[b] = d1 * sDm[lj * P1 + b];
        wz_[b] = d2 * sDm[ll * P1 + b];
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        R gx = R(0), gy = R(0), gz = R(0);
#pragma unroll
        for (int b = 0; b < P1; ++b) {
          gx = fma(wx_[b], sU[v][bx + b], gx);
          gy = fma(wy_[b], sU[v][by + P1 * b], gy);
          gz = fma(wz_[b], sU[v][bz + 16 * b], gz);
        }
        const R al = RAIN && v == V::RR ? al1 : al0;
        sF[0][v][lane] = -al * gx;
        sF[1][v][lane] = -al * gy;
        sF[2][v][lane] = -al * gz;
      }
    }
    __syncthreads();   // the partners' states and fluxes
    constexpr int VH = (NV + 1) / 2;
    SipPoint<R, RAIN> p0, p1;
    R ij[VH], iq[VH];
    // inner face points: lanes 0..31, and 32..63 for the other half of the variables
    const int ji = (lane >> 4) & 1, v0 = (lane >> 5) * (NV - VH);
    const int si = ji ? 1 - dy : 1 - dx;
    const bool inner = WPB > 1 && (ji ? py : px);
    if (act) {
      sip_outer<R, RAIN>(md, f0, l0, Dm, sF, sU, __shfl(al0, f0.n), RAIN ? __shfl(al1, f0.n) : R(0), p0);
      if (!px || !py) {   // wave-uniform
        const R a0 = __shfl(al0, f1.n), a1 = RAIN ? __shfl(al1, f1.n) : R(0);   // (by every lane)
        if (far1) {
          SipLine<R, RAIN> l1;
          sip_line_load<R, RAIN>(U, N, f1, l1);
          sip_outer<R, RAIN>(md, f1, l1, Dm, sF, sU, a0, a1, p1);
        }
      }
      int match;
      const int n = face_node<K, 3>(ji, si, ta, tb, match);
      const R a0 = __shfl(al0, n), a1 = RAIN ? __shfl(al1, n) : a0;
      if (inner) {
        const int ww = w ^ (ji ? BX : 1), nn = n + match;
        const R ct = (R)(ji ? md.sip_tau[1] : md.sip_tau[0]);
#pragma unroll
        for (int i = 0; i < VH; ++i) {
          const int v = v0 + i;
          const R al = RAIN && v == V::RR ? a1 : a0;
          const R d = sU[v][n] - sU_all[ww][v][nn];
          ij[i] = al * (si ? d : -d);
          iq[i] = R(-0.5) * (sF[ji][v][n] + sF_all[ww][ji][v][nn]) - ct * ij[i];
        }
      }
      volume_q3<R, RAIN>(md, li, lj, ll, lane, sF, Rv, sD);
    }
    __syncthreads();   // every read of the viscous fluxes is over
    if (act) {
      // rows of 96 face points: alpha [U] of each variable, then the other term
      R(*sX)[96] = (R(*)[96])&sF[0][0][0];
      const int fp = lane & 15;
      const int r0 = (2 * f0.J + f0.side) * 16 + fp;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        sX[v][r0] = p0.j[v];
        sX[NV + v][r0] = p0.q[v];
      }
      if (far1) {
        const int r1 = (2 * f1.J + 1) * 16 + fp;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          sX[v][r1] = p1.j[v];
          sX[NV + v][r1] = p1.q[v];
        }
      }
      if (inner) {
        const int ri = (2 * ji + si) * 16 + fp;
#pragma unroll
        for (int i = 0; i < VH; ++i) {
          sX[v0 + i][ri] = ij[i];
          sX[NV + v0 + i][ri] = iq[i];
        }
      }
      wave_lds_sync();
      // d_j / w_{i_j} (d_j/2 D[f_j][i_j] alpha [U] + [i_j = f_j] s alpha ({G_j} - tau_j [U]))
      const int idx[3] = {li, lj, ll};
      const int at[3] = {lj + P1 * ll, 32 + li + P1 * ll, 64 + li + P1 * lj};
      R cm[3], cp[3], cq[3];
      int aq[3];
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const R dj = (R)md.two_over_h[j];
        // (the Lobatto weights of k = 3 are 1/6, 5/6, 5/6, 1/6)
        const R kw = (R)md.lift[j][0] * (idx[j] == 0 || idx[j] == K ? R(1) : R(0.2));
        cm[j] = kw * R(0.5) * dj * sDm[idx[j]];
        cp[j] = kw * R(0.5) * dj * sDm[P1 * K + idx[j]];
        cq[j] = idx[j] == 0 ? -kw : (idx[j] == K ? kw : R(0));
        aq[j] = at[j] + (idx[j] == K ? 16 : 0);
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          Rv[v] = fma(cm[j], sX[v][at[j]], Rv[v]);
          Rv[v] = fma(cp[j], sX[v][at[j] + 16], Rv[v]);
          Rv[v] = fma(cq[j], sX[NV + v][aq[j]], Rv[v]);
        }
        asm volatile("" : "+v"(Rv[v]));
        __builtin_amdgcn_sched_barrier(0);
      }
      wave_lds_sync();   // the tiles go on to the fluxes
    }
  }
  if (act) {
    // background table: lane 6 h + f loads field f at height h
    double bgt = 0.0;
    const int bh = lane / kBgStride, bf = lane - kBgStride * bh;
    if (lane < 6 * kBgStride) {
      // height index of the neighbours' face layers below and above (periodic wrap)
      const int zlo = item.hoff + (ez == 0 ? n2 - 1 : ez - 1) * P1 + K;
      const int zhi = item.hoff + (ez == n2 - 1 ? 0 : ez + 1) * P1;
      bgt = a.bgt[(unsigned)(bh < 4 ? izb + bh : (bh == 4 ? zlo : zhi)) * kBgStride + bf];
    }
    // 1. own state
    if constexpr (!SIP) {
#pragma unroll
      for (int v = 0; v < NV; ++v) Uq[v] = ld(U, N, v, g);
    }
    T = ld_f64<R>(auxT, N, g);
    rvs = ld_f64<R>(auxS, N, g);
    if (lane < 6 * kBgStride) (&sB[0][0].x)[lane] = bgt;
    wave_lds_sync();
    if constexpr (SIP) {
#pragma unroll
      for (int v = 0; v < NV; ++v) Uq[v] = sU_all[w][v][lane];
    }

    // 2. point state, fluxes, wave speeds to LDS; the sources
    Pt<R, D, RAIN> q;
    eval_bg<R, D, RAIN>(a, Uq, T, rvs, q3_bg(sB[ll]), q);
    {
      R F[NV];
      flux<R, D, RAIN, 0>(q, F);
#pragma unroll
      for (int v = 0; v < NV; ++v) sF[0][v][lane] = F[v];
      flux<R, D, RAIN, 1>(q, F);
#pragma unroll
      for (int v = 0; v < NV; ++v) sF[1][v][lane] = F[v];
      flux<R, D, RAIN, 2>(q, F);
#pragma unroll
      for (int v = 0; v < NV; ++v) sF[2][v][lane] = F[v];
    }
    if (!SIP && BX == 2 && li == (dx ? 0 : K)) {
#pragma unroll
      for (int v = 0; v < NV; ++v) sI[0][v][lj + P1 * ll] = Uq[v];
    }
    if (!SIP && BY == 2 && lj == (dy ? 0 : K)) {
#pragma unroll
      for (int v = 0; v < NV; ++v) sI[1][v][li + P1 * ll] = Uq[v];
    }
    if (li == 0 || li == K) sL[0][(li ? 16 : 0) + lj + P1 * ll] = wave_speed<R, D, RAIN, 0>(q);
    if (lj == 0 || lj == K) sL[1][(lj ? 16 : 0) + li + P1 * ll] = wave_speed<R, D, RAIN, 1>(q);
    lz = wave_speed<R, D, RAIN, 2>(q);
    sources<R, D, RAIN>(a, Uq, q, Rv);
    // the neighbour traces of the outer faces: in flight until the face pass
    pair_load<R, D, RAIN>(U, auxT, auxS, N, f0.gn, nb0);
  }
  // block-wide (without diffusion the only one): the D-hat table, and the partners'
  // tiles for the faces inside the brick
  __syncthreads();
  if (!act) return;

  // 3. volume term
  volume_q3<R, RAIN>(md, li, lj, ll, lane, sF, Rv, sD);
  wave_lds_sync();   // the volume term has read sF before the faces overwrite it

  // 4. faces: the lifted Lax-Friedrichs correction
  // +-(lift/2)(F + F_n) + (lift/2) Lambda (U_n - U), + on the minus face.
  // (the Lobatto weights are symmetric: both sides lift alike)
  const R hx = R(0.5) * (R)md.lift[0][0], hy = R(0.5) * (R)md.lift[1][0], hz = R(0.5) * (R)md.lift[2][0];
  // (the own traces come across the lanes, so no tile of the state is needed)
  auto own = [&](int v, int n) { return SIP ? sU_all[SIP ? w : 0][v][SIP ? n : 0] : __shfl(Uq[v], n); };
  {
    R Uo[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) Uo[v] = own(v, f0.n);
    q3_outer<R, RAIN>(a, f0, nb0, sF, Uo, __shfl(lz, f0.n), sL, sB, hx, hy, hz);
  }
  if (!px || !py) {   // wave-uniform: the last brick of an odd mesh
    R Uo[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) Uo[v] = own(v, f1.n);   // (by every lane)
    if (far1) {
      pair_load<R, D, RAIN>(U, auxT, auxS, N, f1.gn, nb0);
      q3_outer<R, RAIN>(a, f1, nb0, sF, Uo, R(0), sL, sB, hx, hy, hz);
    }
  }
  // faces inside the brick: both traces and fluxes are in LDS.  Lanes 0..31
  // take the x and y face nodes, lanes 32..63 the same with the other half of
  // the variables (odd counts: one variable twice, the same value).  The
  // correction goes to the node one step inside the element, whose own flux
  // is no longer needed; the face node's flux stays for the partner.
  {
    constexpr int VH = (NV + 1) / 2;
    const int j = (lane >> 4) & 1;         // 0: x, 1: y
    if (WPB > 1 && (j ? py : px)) {
      const int side = j ? 1 - dy : 1 - dx;
      const int ww = w ^ (j ? BX : 1);
      int match;
      const int n = face_node<K, 3>(j, side, ta, tb, match);
      const int nn = n + match;
      const int in = n + (side ? -1 : 1) * (j ? P1 : 1);
      const R lo = sL[j][side * 16 + (lane & 15)], ln = sL_all[ww][j][(1 - side) * 16 + (lane & 15)];
      const bool own = side ? (lo >= ln) : !(ln >= lo);
      const R hl = j ? hy : hx;
      const R kf = side ? -hl : hl;
      const R kj = hl * (own ? lo : ln);
      const int v0 = (lane >> 5) * (NV - VH);
#pragma unroll
      for (int i = 0; i < VH; ++i) {
        const int v = v0 + i, fp = lane & 15;
        const R d = SIP ? sU_all[SIP ? ww : 0][v][SIP ? nn : 0] - sU_all[SIP ? w : 0][v][SIP ? n : 0]
                        : sI_all[SIP ? 0 : ww][j][v][fp] - sI[j][v][fp];
        sF[j][v][in] = fma(kf, sF[j][v][n] + sF_all[ww][j][v][nn], kj * d);
      }
    }
  }
  // operands of the update and the split, fetched while the faces finish
  R U0q[NV];
  if (MODE != 0 && c0 != 0.0) {
#pragma unroll
    for (int v = 0; v < NV; ++v) U0q[v] = ld(U0, N, v, g);
  }
  const Bg bg = q3_bg(sB[ll]);
  wave_lds_sync();

  // 5. face corrections of this node, then the stage epilogue
  const int cx = lane + (px && li == (dx ? 0 : K) ? (dx ? 1 : -1) : 0);
  const int cy = lane + (py && lj == (dy ? 0 : K) ? (dy ? P1 : -P1) : 0);
  if (li == 0 || li == K) {
#pragma unroll
    for (int v = 0; v < NV; ++v) Rv[v] += sF[0][v][cx];
  }
  if (lj == 0 || lj == K) {
#pragma unroll
    for (int v = 0; v < NV; ++v) Rv[v] += sF[1][v][cy];
  }
  if (ll == 0 || ll == K) {
#pragma unroll
    for (int v = 0; v < NV; ++v) Rv[v] += sF[2][v][lane];
  }
  const double dtm = MODE != 0 && dt_m ? dt_m[item.member] : 1.0;
  int iters = 0, bad = 0;
  if constexpr (SIP) {
#pragma unroll
    for (int v = 0; v < NV; ++v) Uq[v] = sU_all[w][v][lane];
  }
  // with diffusion, the new state's element viscosity (Section 3.5) for the
  // next stage: the node shares, then the pairwise sum over the wavefront in
  // the order of sip_alpha_kernel's tree
  constexpr bool ALPHA = SIP && MODE == 2;
  double at[2] = {0.0, 0.0};
  const double wq = ALPHA ? md.J * a.w[li] * a.w[lj] * a.w[ll] : 0.0;
  stage_epilogue<R, D, RAIN, MODE>(a, bg, iz, g, N, Uq, U0q, Rv, T, rvs, out, dtm, c0, c1, c2, oT, oS, flags,
                                   iters, bad, nullptr, nullptr, nullptr, wq, ALPHA ? at : nullptr);
  if (MODE == 2) record_stats(a, seen, iters, bad);
  if constexpr (ALPHA) {
#pragma unroll
    for (int h = 1; h < NP; h <<= 1) {
      at[0] += __shfl_down(at[0], h);
      at[1] += __shfl_down(at[1], h);
    }
    if (lane == 0) {
      a.sip_aK_out[item.eoff + e] = md.sip_pre * sqrt(at[0]);
      a.sip_aK_out[a.etot + item.eoff + e] = md.sip_pre * sqrt(at[1]);
    }
  }
}

}  // namespace dgm
