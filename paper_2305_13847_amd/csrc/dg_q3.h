// Stage kernel for Q3 hexahedra (Lobatto basis): one wavefront per element, a
// 2 x 2 brick (x, y) of elements per block.
//
// A Q3 hexahedron has (3+1)^3 = 64 nodes, so lane n of a wavefront owns node
// n = i + 4 j + 16 l of one element.  Everything that depends on the element
// alone (its coordinates, neighbours, wall flags, offsets) is wave-uniform and
// lives in scalar registers; per-lane indices are bit fields of the lane id.
// Each wavefront works in its own LDS tiles; the block meets once, after the
// fluxes are staged, so that the faces inside the brick take both sides from
// LDS.  With partners on one x and one y side an element has four outer
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
//      F_x, F_y, F_z, U and the wave speeds in LDS; the sources;
//   3. volume term from the LDS lines;
//   4. faces: each lane evaluates one outer neighbour trace (on a slip wall
//      its own, mirrored), forms the Lax-Friedrichs flux with the own trace
//      from LDS, and leaves the lifted correction in LDS; the faces inside
//      the brick need no evaluation;
//   5. every node adds the corrections of its faces, then the stage update,
//      the sponge, the store and the split of the new state (stage_epilogue).
// (FP64: 2 x 1 bricks, five outer faces, the fifth in a quarter pass.)
//
// Bound by HBM traffic and VALU issue together: on 64 x 64 x 32 in FP32 a stage
// moves 0.95 GB (0.66 GB is algorithmic, the rest neighbour data missed by the
// L2s) at 77 % of a copy's rate with the VALU 72 % busy.  Five steps 5.73 ->
// 5.38 ms against one element per wavefront without bricks (1.04 GB per stage,
// four blocks per CU); FP64 31 x 33 x 17, two steps, 580 -> 545 us.
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
// the own trace from LDS; the correction replaces F_J at the own node.
template <typename R, int RAIN>
__device__ __forceinline__ void q3_outer(const KArgs& a, const FaceTask& f, Pair<R, 3, RAIN>& nb,
                                         R (*sF)[Vars<3, RAIN>::NV][64], const R (*sU)[64], const R (*sL)[32],
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
  const R lo = sL[J][f.side * 16 + (int)(threadIdx.x & 15)];
  // Lambda = max over the two sides, ties to the minus side
  const bool own = f.side ? (lo >= ln) : !(ln >= lo);
  const R hl = J == 0 ? hx : (J == 1 ? hy : hz);
  const R kf = f.side ? -hl : hl;
  const R kj = hl * (own ? lo : ln);
#pragma unroll
  for (int v = 0; v < NV; ++v) sF[J][v][f.n] = fma(kf, sF[J][v][f.n] + Fn[v], kj * (nb.nb.U[v] - sU[v][f.n]));
}

__device__ __forceinline__ bool q3_wall(int bc, int c, int n, int side) { return bc == 1 && (side ? c == n - 1 : c == 0); }
// step to the neighbour's coordinate (periodic wrap)
__device__ __forceinline__ int q3_step(int c, int n, int side) {
  return side ? (c == n - 1 ? 1 - n : 1) : (c == 0 ? n - 1 : -1);
}

// FP32: 2 x 2 bricks, 5 wavefronts per SIMD (96 registers; the LDS of five
// blocks fills a CU).  FP64: the tiles are twice as large, and blocks of four
// would leave room for two (8 wavefronts per CU; 31 x 33 x 17, two steps: 609
// us): 2 x 1 bricks, five blocks.
template <typename R>
constexpr int q3_min_waves() { return sizeof(R) == 4 ? 5 : 2; }

template <typename R, int RAIN, int MODE>
__global__ void __launch_bounds__(128 * q3_brick_rows<R>()) __attribute__((amdgpu_waves_per_eu(q3_min_waves<R>())))
rhs_q3_kernel(KArgs a, const R* __restrict__ U, const double* __restrict__ auxT,
              const double* __restrict__ auxS, R* __restrict__ out, const R* __restrict__ U0,
              const double* __restrict__ dt_m, double c0, double c1, double c2, double* __restrict__ oT,
              double* __restrict__ oS, int flags) {
  constexpr int K = 3, P1 = 4, NP = 64, D = 3;
  using V = Vars<D, RAIN>;
  constexpr int NV = V::NV;
  constexpr int BY = q3_brick_rows<R>();
  constexpr int WPB = 2 * BY;   // wavefronts (elements) per block
  // per-wavefront LDS tiles: fluxes of the three directions (later the face
  // corrections), the state, the wave speeds
  __shared__ R sF_all[WPB][D][NV][NP];
  __shared__ R sU_all[WPB][NV][NP];
  __shared__ R sL_all[WPB][D][2 * P1 * P1];   // at the face nodes: side, face node
  // background (KArgs::bgt fields) at the brick's four heights and at the face
  // heights of the neighbours below and above: the same for its elements, and
  // each wavefront writes all of it (the same values) before it reads
  __shared__ double2 sB[6][kBgStride / 2];
  __shared__ R sD[P1 * P1];
  if (threadIdx.x < P1 * P1) sD[threadIdx.x] = (R)a.Dhat[threadIdx.x];

  const ItemWalk walk(a.nbricks, a.walk_rev);
  const int it_ = walk.item(0);
  if (it_ < 0) return;                     // block-uniform
  const int seen = MODE == 2 ? stats_seen(a) : 0;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = (int)(threadIdx.x & 63);
  const Item item = a.bricks[it_];
  const MemberDesc& md = a.mem[item.member];
  R(*sF)[NV][NP] = sF_all[w];
  R(*sU)[NP] = sU_all[w];
  R(*sL)[2 * P1 * P1] = sL_all[w];

  // element (scalar): coordinates, partners inside the brick, outer faces
  const int n0 = item.n[0], n1 = item.n[1], n2 = item.n[2];
  const int b0 = item.bc[0], b1 = item.bc[1], b2 = item.bc[2];
  const int dx = w & 1, dy = w >> 1;       // (BY = 1: dy = 0)
  const int ex = item.c0 + dx, ey = (item.c12 & 0xffff) + dy, ez = item.c12 >> 16;
  const bool act = ex < n0 && ey < n1;     // wave-uniform (odd mesh sizes)
  const bool px = dx == 1 || ex + 1 < n0, py = BY == 2 && (dy == 1 || ey + 1 < n1);
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
  Pair<R, D, RAIN> nb0, nb1;
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
#pragma unroll
    for (int v = 0; v < NV; ++v) Uq[v] = ld(U, N, v, g);
    T = ld(auxT, N, 0, g);
    rvs = ld(auxS, N, 0, g);
    if (lane < 6 * kBgStride) (&sB[0][0].x)[lane] = bgt;
    wave_lds_sync();

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
#pragma unroll
    for (int v = 0; v < NV; ++v) sU[v][lane] = Uq[v];
    if (li == 0 || li == K) sL[0][(li ? 16 : 0) + lj + P1 * ll] = wave_speed<R, D, RAIN, 0>(q);
    if (lj == 0 || lj == K) sL[1][(lj ? 16 : 0) + li + P1 * ll] = wave_speed<R, D, RAIN, 1>(q);
    if (ll == 0 || ll == K) sL[2][(ll ? 16 : 0) + li + P1 * lj] = wave_speed<R, D, RAIN, 2>(q);
#pragma unroll
    for (int v = 0; v < NV; ++v) Rv[v] = R(0);
    sources<R, D, RAIN>(a, Uq, q, Rv);
    // the neighbour traces of the outer faces: in flight until the face pass
    pair_load<R, D, RAIN>(U, auxT, auxS, N, f0.gn, nb0);
    if (BY == 1 && far1) pair_load<R, D, RAIN>(U, auxT, auxS, N, f1.gn, nb1);
  }
  // the only block-wide barrier: the D-hat table, and the partners' tiles for
  // the faces inside the brick
  __syncthreads();
  if (!act) return;

  // 3. volume term
  volume_q3<R, RAIN>(md, li, lj, ll, lane, sF, Rv, sD);
  wave_lds_sync();   // the volume term has read sF before the faces overwrite it

  // 4. faces: the lifted Lax-Friedrichs correction
  // +-(lift/2)(F + F_n) + (lift/2) Lambda (U_n - U), + on the minus face.
  // (the Lobatto weights are symmetric: both sides lift alike)
  const R hx = R(0.5) * (R)md.lift[0][0], hy = R(0.5) * (R)md.lift[1][0], hz = R(0.5) * (R)md.lift[2][0];
  q3_outer<R, RAIN>(a, f0, nb0, sF, sU, sL, sB, hx, hy, hz);
  if (!px || !py) {   // wave-uniform; BY = 2: the last brick of an odd mesh only
    if (far1) {
      if (BY == 2) pair_load<R, D, RAIN>(U, auxT, auxS, N, f1.gn, nb1);
      q3_outer<R, RAIN>(a, f1, nb1, sF, sU, sL, sB, hx, hy, hz);
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
    if (j ? py : px) {
      const int side = j ? 1 - dy : 1 - dx;
      const int ww = w ^ (1 << j);
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
      for (int i = 0; i < VH; ++i)
        sF[j][v0 + i][in] = fma(kf, sF[j][v0 + i][n] + sF_all[ww][j][v0 + i][nn],
                                kj * (sU_all[ww][v0 + i][nn] - sU[v0 + i][n]));
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
  if (flags & kSip) {
#pragma unroll
    for (int v = 0; v < NV; ++v) Rv[v] += ld((const R*)a.sip_out, N, v, g);
  }
  const double dtm = MODE != 0 && dt_m ? dt_m[item.member] : 1.0;
  int iters = 0, bad = 0;
#pragma unroll
  for (int v = 0; v < NV; ++v) Uq[v] = sU[v][lane];
  // with kSipAlpha, the new state's element viscosity (Section 3.5) for the
  // next stage's diffusion: the node shares, then the pairwise sum over the
  // wavefront in the order of sip_alpha_kernel's tree
  double at[2] = {0.0, 0.0};
  const double wq = md.J * a.w[li] * a.w[lj] * a.w[ll];
  stage_epilogue<R, D, RAIN, MODE>(a, bg, iz, g, N, Uq, U0q, Rv, T, rvs, out, dtm, c0, c1, c2, oT, oS, flags,
                                   iters, bad, nullptr, nullptr, nullptr, wq, at);
  if (MODE == 2) record_stats(a, seen, iters, bad);
  if (MODE == 2 && (flags & kSipAlpha)) {
#pragma unroll
    for (int h = 1; h < NP; h <<= 1) {
      at[0] += __shfl_down(at[0], h);
      at[1] += __shfl_down(at[1], h);
    }
    if (lane == 0) {
      a.sip_aK[item.eoff + e] = md.sip_pre * sqrt(at[0]);
      a.sip_aK[a.etot + item.eoff + e] = md.sip_pre * sqrt(at[1]);
    }
  }
}

}  // namespace dgm
