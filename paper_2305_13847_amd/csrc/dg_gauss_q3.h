// Right-hand side / stage kernel of the Gauss basis on Q3 hexahedra: the method
// of dg_gauss.h (its trace buffers included) on the bricks of dg_q3.h.
//
// One wavefront per element, a 2 x 2 brick (x, y) per block (Brick).
// Everything that depends on the element alone is wave-uniform.  Of an
// element's 96 face points the 64 on the brick's outside are one pass of its
// lanes: the own trace from its LDS tiles, the neighbour's from the trace
// buffer.  A face inside the brick is evaluated once, for both elements: a
// lane per side and point takes that side's trace and flux, the pair exchanges
// them by a shuffle.  Such faces neither read nor write the trace buffers.
//
// Bound by HBM traffic and VALU issue together: a stage moves 11.7 KB per
// element in FP32 (14.5 with the block kernel of dg_gauss.h, which serves the
// other orders), in 5 instead of 6 wavefront passes over face points per four
// elements, and its sources, index work and neighbour loads come before the
// volume term, which is what frees the registers for 4 wavefronts per SIMD.
// 48 x 48 x 24 elements with rain, two SSPRK(4,3) steps: FP32 2.25 -> 1.66 ms,
// FP64 4.35 -> 2.59; 21 x 21 x 11: 291 -> 228 us and 423 -> 320; 5 x 4 x 3
// (launches and one wave's chain): 137 -> 100 and 139 -> 107.
#pragma once
#include "dg_gauss.h"
#include "dg_q3.h"

namespace dgm {

// Line through face point (ta, tb) of direction J: first node and stride.
__device__ __forceinline__ void gq3_line(int J, int ta, int tb, int& n0, int& str) {
  n0 = (J == 0 ? 4 * ta : ta) + (J == 2 ? 4 * tb : 16 * tb);
  str = J == 0 ? 1 : (J == 1 ? 4 : 16);
}

// Trace of U', T and rho_v at side `side` of the line, from an element's tiles.
// The face passes and the trace writer share this code, so both sides of a
// face see the same bits.
template <typename R, int RAIN>
__device__ __forceinline__ void gq3_trace(int n0, int str, int side, const R (*sU)[64], const double* sT,
                                          const double* sRv, const R (*sW)[4], const double (*sWd)[4], R* Ut,
                                          double& Tt, double& Rvt) {
  constexpr int NV = Vars<3, RAIN>::NV;
#pragma unroll
  for (int v = 0; v < NV; ++v) Ut[v] = R(0);
  Tt = 0.0;
  Rvt = 0.0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int nd = n0 + i * str;
    const R w = sW[side][i];
    const double wd = sWd[side][i];
#pragma unroll
    for (int v = 0; v < NV; ++v) Ut[v] = fma(w, sU[v][nd], Ut[v]);
    Tt = fma(wd, sT[nd], Tt);
    Rvt = fma(wd, sRv[nd], Rvt);
  }
}

// One side of a face point: normal flux and wave speed.
template <typename R, int RAIN>
__device__ __forceinline__ void gq3_side(const KArgs& a, int J, const R* Ut, double T, double rv, const Bg& b, R* F,
                                         R& l) {
  Pt<R, 3, RAIN> q;
  eval_core<R, 3, RAIN>(a, Ut, T, rv, rv, b.rd, b.rm, RAIN ? b.rr : 0.0, b.p, b.Ep, q);
  const R uj = J == 0 ? q.u[0] : (J == 1 ? q.u[1] : q.u[2]);
  flux_sel<R, 3, RAIN>(q, J, uj, F);
  l = fabs(uj) + q.cm;
  if (RAIN) l += J == 2 ? fabs(q.vr) : R(0);
}

// An outer face task: direction, side, point, the neighbour's entry in the
// trace buffers and the background rows of both sides.
struct GTask {
  int J, side, fp, bo, bn;
  bool wall;
  unsigned rn;   // neighbour's face point: element * 96 + face point
};

__device__ __forceinline__ GTask gq3_task(int J, int side, int fp, bool wall, int en) {
  GTask t;
  t.J = J;
  t.side = side;
  t.fp = fp;
  t.wall = wall;
  t.bo = J == 2 ? 4 + side : fp >> 2;
  t.bn = J == 2 && !wall ? 6 + side : t.bo;
  t.rn = (unsigned)en * 96u + (unsigned)((2 * J + 1 - side) * 16 + fp);
  return t;
}

// The trace of the element's tiles at an outer face point, to the output buffers.
template <typename R, int RAIN>
__device__ __forceinline__ void gq3_write(const KArgs& a, const GTask& t, int e, unsigned ntr, const R (*sU)[64],
                                          const double* sT, const double* sRv, const R (*sW)[4],
                                          const double (*sWd)[4]) {
  constexpr int NV = Vars<3, RAIN>::NV;
  int l0, str;
  gq3_line(t.J, t.fp & 3, t.fp >> 2, l0, str);
  R Ut[NV];
  double Tt, Rvt;
  gq3_trace<R, RAIN>(l0, str, t.side, sU, sT, sRv, sW, sWd, Ut, Tt, Rvt);
  const unsigned at = (unsigned)e * 96u + (unsigned)((2 * t.J + t.side) * 16 + t.fp);
#pragma unroll
  for (int v = 0; v < NV; ++v) st((R*)a.tr_u_out, ntr, v, at, Ut[v]);
  st(a.tr_a_out, ntr, 0, at, Tt);
  st(a.tr_a_out, ntr, 1, at, Rvt);
}

template <typename R, int RAIN>
struct GNb {
  R U[Vars<3, RAIN>::NV];
  double T, rv;
};

template <typename R, int RAIN>
__device__ __forceinline__ void gq3_load(const KArgs& a, const GTask& t, unsigned ntr, GNb<R, RAIN>& n) {
#pragma unroll
  for (int v = 0; v < Vars<3, RAIN>::NV; ++v) n.U[v] = ld((const R*)a.tr_u_in, ntr, v, t.rn);
  n.T = ld(a.tr_a_in, ntr, 0, t.rn);
  n.rv = ld(a.tr_a_in, ntr, 1, t.rn);
}

// Flux of an outer face point (normal +e_J) into sX[v][face point].
template <typename R, int RAIN>
__device__ __forceinline__ void gq3_outer(const KArgs& a, const GTask& t, GNb<R, RAIN>& nb, const R (*sU)[64],
                                          const double* sT, const double* sRv, const R (*sW)[4],
                                          const double (*sWd)[4], const double2 (*sB)[3], R (*sX)[96]) {
  using V = Vars<3, RAIN>;
  constexpr int NV = V::NV;
  int n0, str;
  gq3_line(t.J, t.fp & 3, t.fp >> 2, n0, str);
  R Uo[NV], Fo[NV], Fn[NV], lo, ln;
  double To, Rvo;
  gq3_trace<R, RAIN>(n0, str, t.side, sU, sT, sRv, sW, sWd, Uo, To, Rvo);
  gq3_side<R, RAIN>(a, t.J, Uo, To, Rvo, q3_bg(sB[t.bo]), Fo, lo);
  if (t.wall) {
    // slip wall: the own trace mirrored
#pragma unroll
    for (int v = 0; v < NV; ++v) nb.U[v] = Uo[v];
#pragma unroll
    for (int i = 0; i < 3; ++i) nb.U[V::M0 + i] = i == t.J ? -Uo[V::M0 + i] : Uo[V::M0 + i];
    nb.T = To;
    nb.rv = Rvo;
  }
  gq3_side<R, RAIN>(a, t.J, nb.U, nb.T, nb.rv, q3_bg(sB[t.bn]), Fn, ln);
  // Lambda = max over the two sides, ties to the minus side: both elements take the
  // same one, also where a side's speed is not a number (a trace with T < 0)
  const R lm = t.side ? lo : ln, lp = t.side ? ln : lo;
  const R hL = R(0.5) * (lm >= lp ? lm : lp);
  const int at = (2 * t.J + t.side) * 16 + t.fp;
#pragma unroll
  for (int v = 0; v < NV; ++v)
    sX[v][at] = R(0.5) * (Fo[v] + Fn[v]) + hL * (t.side ? Uo[v] - nb.U[v] : nb.U[v] - Uo[v]);
}

// One direction's share of the volume term: the point's flux to the wavefront's
// tile (rows of 64 nodes), then R_v += (2/h_J) sum_b Dhat[i_J][b] F_J,v(node b on
// the lane's J-line).  `i`: the lane's index along J, `str`: the line's stride.
template <typename R, int RAIN, int J>
__device__ __forceinline__ void gq3_volume(const MemberDesc& md, const Pt<R, 3, RAIN>& q, int i, int lane,
                                           R (*sF)[64], const R* sD, R* Rv) {
  constexpr int NV = Vars<3, RAIN>::NV, str = J == 0 ? 1 : (J == 1 ? 4 : 16);
  R F[NV];
  flux<R, 3, RAIN, J>(q, F);
#pragma unroll
  for (int v = 0; v < NV; ++v) sF[v][lane] = F[v];
  wave_lds_sync();
  const R s = (R)md.two_over_h[J];
  const int b0 = lane - i * str;
  R d[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) d[b] = sD[i * 4 + b];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    R x = d[0] * sF[v][b0];
#pragma unroll
    for (int b = 1; b < 4; ++b) x += d[b] * sF[v][b0 + b * str];
    Rv[v] += s * x;
    asm volatile("" : "+v"(Rv[v]));   // (not sunk to its use: the LDS values would stay in registers)
  }
  wave_lds_sync();
}

template <typename R>
constexpr int gq3_min_waves() { return sizeof(R) == 4 ? 4 : 3; }

// Directions of the volume term in LDS at once.  FP32: all three (one at a time,
// 24 instead of 34 KB a brick, 1.68 -> 1.71 ms at the same 4 wavefronts per SIMD,
// and 1.82 at 5, where 96 registers spill; 48 x 48 x 24, two steps).  FP64: one,
// which makes room for a third brick per CU (2.93 -> 2.59 ms).
template <typename R>
constexpr int gq3_tiles() { return sizeof(R) == 4 ? 3 : 1; }

template <typename R, int RAIN, int MODE, int BX, int BY>
__global__ void __launch_bounds__(64 * BX * BY) __attribute__((amdgpu_waves_per_eu(gq3_min_waves<R>())))
rhs_gauss_q3_kernel(KArgs a, const R* __restrict__ U, const double* __restrict__ auxT,
                    const double* __restrict__ auxS, R* __restrict__ out, const R* __restrict__ U0,
                    const double* __restrict__ dt_m, double c0, double c1, double c2, double* __restrict__ oT,
                    double* __restrict__ oS, int flags) {
  constexpr int P1 = 4, NP = 64, D = 3, WPB = BX * BY;
  using V = Vars<D, RAIN>;
  constexpr int NV = V::NV;
  constexpr int TILES = gq3_tiles<R>();
  constexpr int XF = BX == 2 ? BY : 0, YF = BY == 2 ? BX : 0;   // x and y faces inside the brick
  // per element: the fluxes of TILES directions (after the volume term those of its
  // outer face points), the state, T and rho_v
  __shared__ R sF_all[WPB][TILES == 3 ? D * NV * NP : NV * 96];
  __shared__ R sU_all[WPB][NV][NP];
  __shared__ double sT_all[WPB][NP], sRv_all[WPB][NP];
  __shared__ R sI[NV][64];                 // fluxes of the faces inside the brick, 16 points each
  // background: the four node heights, the faces below and above of this row
  // of elements, and their outer sides
  __shared__ double2 sB[8][kBgStride / 2];
  __shared__ R sD[P1 * P1], sW[2][P1], sK[D][P1][2];
  __shared__ double sWd[2][P1];

  const ItemWalk walk(a.nbricks, a.walk_rev);
  const int it_ = walk.item(0);
  if (it_ < 0) return;                     // block-uniform
  const int seen = MODE == 2 ? stats_seen(a) : 0;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = (int)(threadIdx.x & 63);
  const Item item = a.bricks[it_];
  const MemberDesc& md = a.mem[item.member];
  // (every wavefront writes the tables that it reads before the block meets)
  if (lane < P1 * P1) sD[lane] = (R)a.Dhat[lane];
  if (threadIdx.x < 2 * P1) {
    const int s = threadIdx.x >> 2, i = threadIdx.x & 3;
    const double l = s ? a.gl_p[i] : a.gl_m[i];
    sWd[s][i] = l;
    sW[s][i] = (R)l;
  }
  if (threadIdx.x < 2 * D * P1) {
    const int j = threadIdx.x >> 3, i = (threadIdx.x >> 1) & 3, s = threadIdx.x & 1;
    sK[j][i][s] = (R)(md.two_over_h[j] * (s ? a.lift_p[i] : a.lift_m[i]));
  }
  R(*sU)[NP] = sU_all[w];
  R(*sX)[96] = (R(*)[96])sF_all[w];
  R(*sF)[NP] = (R(*)[NP])sF_all[w];

  // element (scalar): coordinates, partners inside the brick, outer faces
  const int n0 = item.n[0], n1 = item.n[1], n2 = item.n[2];
  const int b0 = item.bc[0], b1 = item.bc[1], b2 = item.bc[2];
  const Brick<BX, BY> br(item, w);
  const int dx = br.dx, dy = br.dy, ex = br.ex, ey = br.ey, ez = br.ez;
  const bool act = br.act, px = br.px, py = br.py;   // wave-uniform
  const int e = item.eoff + item.e0 + dx + dy * n0;
  const unsigned N = a.nnodes, ntr = (unsigned)a.etot * 96u;
  const unsigned g = (unsigned)e * NP + lane;
  const int li = lane & 3, lj = (lane >> 2) & 3, ll = lane >> 4;
  const int izb = item.hoff + ez * P1;
  const int iz = izb + ll;
  // outer face tasks, 16 lanes per face: x and y on the side away from the
  // brick, z below and above; far sides (f1): lanes 0..15 x, 16..31 y
  const int tf = lane >> 4, fp = lane & 15;
  const bool wx = q3_wall(b0, ex, n0, dx), wy = q3_wall(b1, ey, n1, dy);
  const bool wz0 = q3_wall(b2, ez, n2, 0), wz1 = q3_wall(b2, ez, n2, 1);
  const int nn01 = n0 * n1;
  const int qx = q3_step(ex, n0, dx), qy = q3_step(ey, n1, dy) * n0;
  const int qz0 = q3_step(ez, n2, 0) * nn01, qz1 = q3_step(ez, n2, 1) * nn01;
  const GTask f0 = gq3_task(tf < 2 ? tf : 2, tf == 0 ? dx : (tf == 1 ? dy : tf - 2), fp,
                            tf == 0 ? wx : (tf == 1 ? wy : (tf == 2 ? wz0 : wz1)),
                            e + (tf == 0 ? qx : (tf == 1 ? qy : (tf == 2 ? qz0 : qz1))));
  // (formed where it is used: a brick of an odd mesh alone needs it)
  auto far = [&]() {
    return gq3_task(tf & 1, 1, fp, (tf & 1) ? q3_wall(b1, ey, n1, 1) : q3_wall(b0, ex, n0, 1),
                    e + ((tf & 1) ? q3_step(ey, n1, 1) * n0 : q3_step(ex, n0, 1)));
  };
  const bool far1 = (tf == 0 && !px) || (tf == 1 && !py);

  R Uq[NV], Rv[NV];
  double T = 300.0, rvs = 0.0;
  GNb<R, RAIN> nb0;
  if (act) {
    // background table: lane 6 h + f loads field f (KArgs::bgt) of row h
    const int bh = lane / kBgStride, bf = lane - kBgStride * bh;
    double bgt = 0.0;
    if (lane < 8 * kBgStride) {
      if (bh < 4) {
        bgt = a.bgt[(unsigned)(izb + bh) * kBgStride + bf];
      } else {
        const int r0 = item.hoff / P1;
        const int row = bh < 6 ? ez : (bh == 6 ? (ez == 0 ? n2 - 1 : ez - 1) : (ez == n2 - 1 ? 0 : ez + 1));
        const int at = 2 * (r0 + row) + (bh < 6 ? bh - 4 : 7 - bh);
        const int src = bf == 2 ? 4 : (bf == 3 || bf == 5 ? 3 : (bf == 4 ? 2 : bf));
        bgt = a.bgf[src * a.bgf_n + at];
        if (bf == 3) bgt += a.bgf[4 * a.bgf_n + at];
      }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) Uq[v] = ld(U, N, v, g);
    T = ld(auxT, N, 0, g);
    rvs = ld(auxS, N, 0, g);
    // (every wavefront of the brick writes the same table before it reads)
    if (lane < 8 * kBgStride) (&sB[0][0].x)[lane] = bgt;
    wave_lds_sync();
    Pt<R, D, RAIN> q;
    const Bg b = q3_bg(sB[ll]);
    eval_bg<R, D, RAIN>(a, Uq, T, rvs, b, q);
    if constexpr (TILES == 3) {
      R F[NV];
      flux<R, D, RAIN, 0>(q, F);
#pragma unroll
      for (int v = 0; v < NV; ++v) sF[v][lane] = F[v];
      flux<R, D, RAIN, 1>(q, F);
#pragma unroll
      for (int v = 0; v < NV; ++v) sF[NV + v][lane] = F[v];
      flux<R, D, RAIN, 2>(q, F);
#pragma unroll
      for (int v = 0; v < NV; ++v) sF[2 * NV + v][lane] = F[v];
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) sU[v][lane] = Uq[v];
    sT_all[w][lane] = T;
    sRv_all[w][lane] = fmin(rvs, b.rm + (double)Uq[V::RM]);
#pragma unroll
    for (int v = 0; v < NV; ++v) Rv[v] = R(0);
    sources<R, D, RAIN>(a, Uq, q, Rv);
    // the neighbours' traces: in flight until the face pass
    gq3_load<R, RAIN>(a, f0, ntr, nb0);
    if constexpr (TILES == 1) {
      gq3_volume<R, RAIN, 0>(md, q, li, lane, sF, sD, Rv);
      gq3_volume<R, RAIN, 1>(md, q, lj, lane, sF, sD, Rv);
      gq3_volume<R, RAIN, 2>(md, q, ll, lane, sF, sD, Rv);
    }
  }
  __syncthreads();   // the small tables, and the partners' tiles
  if (act) {
    if constexpr (TILES == 3) {
      volume_q3<R, RAIN>(md, li, lj, ll, lane, (R(*)[NV][NP])sF_all[w], Rv, sD);
      wave_lds_sync();   // the volume term has read sF before the face fluxes replace it
    }
    gq3_outer<R, RAIN>(a, f0, nb0, sU, sT_all[w], sRv_all[w], sW, sWd, sB, sX);
    if (!px || !py) {   // wave-uniform: the last brick of an odd mesh
      if (far1) {
        const GTask f1 = far();
        gq3_load<R, RAIN>(a, f1, ntr, nb0);
        gq3_outer<R, RAIN>(a, f1, nb0, sU, sT_all[w], sRv_all[w], sW, sWd, sB, sX);
      }
    }
    // the faces inside the brick, one per wavefront: the x faces of its rows, then
    // the y faces of its columns.  Lanes 0..15 the lower
    // element's side, 16..31 the upper's.
    const int J = WPB == 4 ? w >> 1 : (BX == 2 ? 0 : 1), k = WPB == 4 ? w & 1 : w;
    const int cx = item.c0 + (J ? k : 1), cy = (item.c12 & 0xffff) + (J ? 1 : k);
    if ((WPB == 4 || w < XF + YF) && cx < n0 && cy < n1) {
      const int up = (lane >> 4) & 1;
      const int ww = J ? k + BX * up : BX * k + up;
      int l0, str;
      gq3_line(J, fp & 3, fp >> 2, l0, str);
      R Uo[NV], Fo[NV], lo;
      double To, Rvo;
      gq3_trace<R, RAIN>(l0, str, 1 - up, sU_all[ww], sT_all[ww], sRv_all[ww], sW, sWd, Uo, To, Rvo);
      gq3_side<R, RAIN>(a, J, Uo, To, Rvo, q3_bg(sB[fp >> 2]), Fo, lo);
      const R ln = __shfl_xor(lo, 16);
      const R hL = R(0.5) * (lo >= ln ? lo : ln);   // (lanes 0..15: the minus side is their own)
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const R Fn = __shfl_xor(Fo[v], 16), Un = __shfl_xor(Uo[v], 16);
        const R Fs = R(0.5) * (Fo[v] + Fn) + hL * (Uo[v] - Un);
        if (lane < 16) sI[v][16 * w + fp] = Fs;
      }
    }
  }
  R U0q[NV];
  if (MODE != 0 && act && c0 != 0.0) {
#pragma unroll
    for (int v = 0; v < NV; ++v) U0q[v] = ld(U0, N, v, g);
  }
  __syncthreads();   // the inner fluxes; every read of the state tiles is over
  if (!act) return;

  // lifting: + l_i(-1)/w_i F*(minus face) - l_i(+1)/w_i F*(plus face)
  {
    // inner face numbers of this element: x face of row dy, y face of column dx
    const R* const xm = dx == 1 ? &sI[0][16 * dy] : &sX[0][0];
    const R* const xp = dx == 0 && px ? &sI[0][16 * dy] : &sX[0][16];
    const R* const ym = dy == 1 ? &sI[0][16 * (XF + dx)] : &sX[0][32];
    const R* const yp = dy == 0 && py ? &sI[0][16 * (XF + dx)] : &sX[0][48];
    const int sxm = dx == 1 ? 64 : 96, sxp = dx == 0 && px ? 64 : 96;   // their rows
    const int sym = dy == 1 ? 64 : 96, syp = dy == 0 && py ? 64 : 96;
    const int fx = lj + P1 * ll, fy = li + P1 * ll, fz = li + P1 * lj;
    const R kxm = sK[0][li][0], kxp = sK[0][li][1], kym = sK[1][lj][0], kyp = sK[1][lj][1];
    const R kzm = sK[2][ll][0], kzp = sK[2][ll][1];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      Rv[v] += kxm * xm[v * sxm + fx] - kxp * xp[v * sxp + fx];
      Rv[v] += kym * ym[v * sym + fy] - kyp * yp[v * syp + fy];
      Rv[v] += kzm * sX[v][64 + fz] - kzp * sX[v][80 + fz];
    }
  }
  const double dtm = MODE != 0 && dt_m ? dt_m[item.member] : 1.0;
  int iters = 0, bad = 0;
#pragma unroll
  for (int v = 0; v < NV; ++v) Uq[v] = sU[v][lane];
  T = sT_all[w][lane];
  const Bg bg = q3_bg(sB[ll]);
  if constexpr (MODE == 2) {
    R Unew[NV];
    double Tnew = 300.0, Snew = 0.0;
    stage_epilogue<R, D, RAIN, MODE>(a, bg, iz, g, N, Uq, U0q, Rv, T, rvs, out, dtm, c0, c1, c2, oT, oS, flags, iters,
                                     bad, Unew, &Tnew, &Snew);
    record_stats(a, seen, iters, bad);
    // the traces of the new state at the outer faces, for the next stage
#pragma unroll
    for (int v = 0; v < NV; ++v) sU[v][lane] = Unew[v];
    sT_all[w][lane] = Tnew;
    sRv_all[w][lane] = fmin(Snew, bg.rm + (double)Unew[V::RM]);
    wave_lds_sync();
    gq3_write<R, RAIN>(a, f0, e, ntr, sU, sT_all[w], sRv_all[w], sW, sWd);
    if (!px || !py) {
      if (far1) gq3_write<R, RAIN>(a, far(), e, ntr, sU, sT_all[w], sRv_all[w], sW, sWd);
    }
  } else {
    stage_epilogue<R, D, RAIN, MODE>(a, bg, iz, g, N, Uq, U0q, Rv, T, rvs, out, dtm, c0, c1, c2, oT, oS, flags, iters,
                                     bad);
  }
}

// Traces of a state that no stage produced, at the outer faces of the bricks.  The
// block kernel (gauss_trace_kernel) wrote all 96 face points of an element, those
// inside a brick for nothing: 48 x 48 x 24 in FP32 with rain 74 -> 62 us.
template <typename R, int RAIN, int BX, int BY>
__global__ void __launch_bounds__(64 * BX * BY)
gauss_q3_trace_kernel(KArgs a, const R* __restrict__ U, const double* __restrict__ auxT,
                      const double* __restrict__ auxS) {
  using V = Vars<3, RAIN>;
  constexpr int NV = V::NV, NP = 64, WPB = BX * BY;
  __shared__ R sU_all[WPB][NV][NP];
  __shared__ double sT_all[WPB][NP], sRv_all[WPB][NP];
  __shared__ R sW[2][4];
  __shared__ double sWd[2][4];
  const int it_ = ItemWalk(a.nbricks).item(0);
  if (it_ < 0) return;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = (int)(threadIdx.x & 63);
  const Item item = a.bricks[it_];
  const Brick<BX, BY> br(item, w);
  const int dx = br.dx, dy = br.dy, n0 = item.n[0], ez = br.ez;
  const bool px = br.px, py = br.py;
  if (!br.act) return;                     // wave-uniform; the block never meets
  const int e = item.eoff + item.e0 + dx + dy * n0;
  const unsigned N = a.nnodes, ntr = (unsigned)a.etot * 96u, g = (unsigned)e * NP + lane;
  R Uq[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) Uq[v] = ld(U, N, v, g);
  const double T = ld(auxT, N, 0, g), rvs = ld(auxS, N, 0, g);
  const double rm = a.bg_rm[item.hoff + ez * 4 + (lane >> 4)];
  // (every wavefront writes the weights that it reads)
  if (lane < 8) {
    const int s = lane >> 2, i = lane & 3;
    const double l = s ? a.gl_p[i] : a.gl_m[i];
    sWd[s][i] = l;
    sW[s][i] = (R)l;
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) sU_all[w][v][lane] = Uq[v];
  sT_all[w][lane] = T;
  sRv_all[w][lane] = fmin(rvs, rm + (double)Uq[V::RM]);
  wave_lds_sync();
  // (the writer needs direction, side and point of a task only)
  const int tf = lane >> 4, fp = lane & 15;
  gq3_write<R, RAIN>(a, gq3_task(tf < 2 ? tf : 2, tf == 0 ? dx : (tf == 1 ? dy : tf - 2), fp, false, e), e, ntr,
                     sU_all[w], sT_all[w], sRv_all[w], sW, sWd);
  if ((tf == 0 && !px) || (tf == 1 && !py))
    gq3_write<R, RAIN>(a, gq3_task(tf & 1, 1, fp, false, e), e, ntr, sU_all[w], sT_all[w], sRv_all[w], sW, sWd);
}

}  // namespace dgm
