// Shared host/device definitions of libdgmoist: kernel argument blocks and the
// per-member mesh descriptors of a (possibly batched) handle.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dgm {

constexpr int kMaxOrder = 7;     // 2D; 3D kernels are instantiated up to 4
constexpr int kMaxP1 = kMaxOrder + 1;

// Status words of a handle (KArgs::stats).  Blocks spread their iteration
// maxima over kStatSlots lines: with a single word, the first launch on a new
// handle (or after a reset) waited about 400 us for its wavefronts' atomics.
constexpr int kStatSlots = 64, kStatStride = 32;
constexpr int kStatsWords = kStatStride * (1 + kStatSlots);

inline unsigned stats_max_iters(const unsigned* w) {
  unsigned m = 0;
  for (int s = 0; s < kStatSlots; ++s) {
    const unsigned v = w[kStatStride * (1 + s)];
    if (v > m) m = v;
  }
  return m;
}

constexpr int kBgStride = 6;

// One ensemble member: a structured box.  Elements of all members are
// concatenated; eoff is this member's first global element.
struct MemberDesc {
  int n[3];             // elements per axis (n[2] = 1 in 2D)
  int bc[3];            // 0 periodic, 1 slip wall
  double two_over_h[3]; // 2 / h_j
  double J;             // element Jacobian prod_j h_j / 2
  double face_J[3];     // face Jacobian for a face normal to axis j
  double lift[3][2];    // (2 / h_j) / w_0 and (2 / h_j) / w_K: face-to-node lifting
  long long eoff;       // first global element
  int ne;               // elements of this member
  int hoff;             // first background index (n_z (k+1) entries)
  // artificial diffusion: gamma 0.5 h^(1-d/2), the penalty sigma k^2 / h_j,
  // the vertices per axis and the first vertex of this member
  double sip_pre;
  double sip_tau[3];
  int nvx[3];
  long long voff;
};

// A work item: EPB consecutive elements of one member, starting at element e0
// with element coordinates (c0, c1, c2) packed as c12 = c1 + (c2 << 16).  It
// carries what addresses depend on (the member's mesh and offsets), one 64-byte
// scalar load: read through the member table these values were a second and
// third scalar round trip before a wavefront's first vector load, half of its
// life in a 64-member ensemble.
struct alignas(64) Item {
  int member;
  int e0;
  int c0;
  int c12;
  int n[3];    // the member's elements per axis,
  int bc[3];   // boundary types,
  int ne;      // elements,
  int eoff;    // first global element
  int hoff;    // and first background index
};

// Everything the kernels need besides the state arrays.
struct KArgs {
  // thermodynamics (Section 2; appendix table)
  double g, cvd, cvv, cl, Rd, Rv, Tref;
  double Lp;                       // L_ref - R_v T_ref
  double am1, b, inv_Tref, C0;     // rho_vs(T) = C0 exp(am1 ln(T/T_ref) + b (1/T_ref - 1/T))
  double vr_const, vr_pref, q_au;  // terminal speed, COSMO prefactor, autoconversion threshold
  int rain, vr_mode;
  double rtol;
  int maxit;
  int closed;                      // the split may solve in closed form (kEstIters)
  // nodal tables of the basis (Lobatto, or Gauss for basis 1):
  // Dhat[i*(k+1)+a] = w_a D_ai / w_i, weights w
  double Dhat[kMaxP1 * kMaxP1];
  double w[kMaxP1];
  // basis 1 (Gauss nodes): traces l_i(-1), l_i(+1) of the Lagrange basis and
  // the lifting weights l_i(-+1) / w_i
  int basis;
  double gl_m[kMaxP1], gl_p[kMaxP1];
  double lift_m[kMaxP1], lift_p[kMaxP1];
  // basis 1: background traces on the horizontal faces, bgf[f * bgf_n + 2 r + s]
  // for field f = (rho_d, rho_m, rho_r, E, p), element row r of the
  // concatenated columns (hoff / (k+1) + ez) and side s (0 bottom, 1 top)
  const double* bgf;
  int bgf_n;
  // basis 1: face traces of the stage state (read) and of the new state
  // (written by MODE 2): U' at tr_u[(v * etot + e) * NFE + f], T and rho_v at
  // tr_a[(c * etot + e) * NFE + f] for face point f of element e
  const void* tr_u_in;
  const double* tr_a_in;
  void* tr_u_out;
  double* tr_a_out;
  // artificial diffusion (Lobatto basis): collocation derivative matrix
  // Dm[a*(k+1)+i] = l_i'(x_a), Lobatto nodes, per-element viscosity aK[2][e],
  // vertex means av[2][vertex] and the diffusive tendency (state layout)
  double Dm[kMaxP1 * kMaxP1];
  double xn[kMaxP1];
  double* sip_aK;
  double* sip_aK_out;              // (Q3 hexahedra) the new state's, written by MODE 2
  double* sip_av;
  void* sip_out;
  long long nvert;
  // members and work items (member, first element) of EPB elements each
  const MemberDesc* mem;
  const Item* items;
  int nitems;
  int epb;                         // elements per work item
  const Item* bricks;              // Q3 hexahedra: bricks (first element and its coordinates)
  int nbricks;
  int brick[2];                    // their elements along x and y
  int nmembers;
  long long etot;                  // elements of all members
  unsigned nnodes;                 // nodes of all members: the stride between variables
  // background per vertical node index, concatenated over members
  const double* bg_rd;
  const double* bg_rm;
  const double* bg_rr;
  const double* bg_E;
  const double* bg_p;
  // the same per index as kBgStride consecutive values (rho_d, rho_m, p, E + p,
  // rho_r, E): a node's background is two or three 16-byte loads of one address
  const double* bgt;
  // sponge blending factor per vertical node index (nullptr: no sponge)
  const double* sponge;
  // status words: [1] non-converged, [2] invalid; the iteration maximum in
  // kStatSlots words of a cache line each (stat_slot), the host takes the largest
  unsigned* stats;
  // stage kernels: walk the work items from the last one (every other stage,
  // so a stage starts on the data the previous one wrote last)
  int walk_rev;
};

}  // namespace dgm
