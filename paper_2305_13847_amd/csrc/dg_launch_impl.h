// Definitions of the launchers of dg_launch.h (included by the translation
// units that instantiate them).
#pragma once
#include <type_traits>
#include "dg_launch.h"
#include "dg_q3.h"
#include "dg_gauss.h"
#include "dg_gauss_q3.h"
#include "dg_sip.h"
#include "dg_vjp.h"

namespace dgm {

template <typename F>
bool dispatch_shape(int K, int D, int rain, F&& f) {
#define DGM_CASE(k, d, r)                                                         \
  if (K == k && D == d && rain == r) {                                            \
    f(std::integral_constant<int, k>{}, std::integral_constant<int, d>{},         \
      std::integral_constant<int, r>{});                                          \
    return true;                                                                  \
  }
  DGM_CASE(1, 2, 0) DGM_CASE(1, 2, 1) DGM_CASE(1, 3, 0) DGM_CASE(1, 3, 1)
  DGM_CASE(2, 2, 0) DGM_CASE(2, 2, 1) DGM_CASE(2, 3, 0) DGM_CASE(2, 3, 1)
  DGM_CASE(3, 2, 0) DGM_CASE(3, 2, 1) DGM_CASE(3, 3, 0) DGM_CASE(3, 3, 1)
  DGM_CASE(4, 2, 0) DGM_CASE(4, 2, 1) DGM_CASE(4, 3, 0) DGM_CASE(4, 3, 1)
  // 2D only above 4: a 3D element of order >= 5 has more nodes than a block
  DGM_CASE(5, 2, 0) DGM_CASE(5, 2, 1) DGM_CASE(6, 2, 0) DGM_CASE(6, 2, 1)
  DGM_CASE(7, 2, 0) DGM_CASE(7, 2, 1)
#undef DGM_CASE
  return false;
}

// f(BX, BY) with the brick of the handle
template <typename F>
void dispatch_brick(const KArgs& a, F&& f) {
  constexpr std::integral_constant<int, 1> one{};
  constexpr std::integral_constant<int, 2> two{};
  if (a.brick[0] == 2 && a.brick[1] == 2) f(two, two);
  else if (a.brick[0] == 2) f(two, one);
  else if (a.brick[1] == 2) f(one, two);
  else f(one, one);
}

template <typename R>
bool LaunchPoint<R>::split(const KArgs& a, LaunchCfg lc, int K, int D, int rain, int item0, int nitems,
    const void* U, const double* guess, double* oT, double* o1, double* o2, int api,
    hipStream_t s) {
  if (nitems <= 0) return true;
  return dispatch_shape(K, D, rain, [&](auto k, auto d, auto r) {
    constexpr int K_ = decltype(k)::value, D_ = decltype(d)::value, R_ = decltype(r)::value;
    // one block per work item whatever the persistence setting (the split
    // kernel has no item loop)
    dim3 grid(grid_for_items(nitems)), block(lc.threads);
    if (api)
      hipLaunchKernelGGL((split_kernel<R, K_, D_, R_, 1>), grid, block, 0, s, a, item0, nitems,
                         (const R*)U, guess, oT, o1, o2);
    else
      hipLaunchKernelGGL((split_kernel<R, K_, D_, R_, 0>), grid, block, 0, s, a, item0, nitems,
                         (const R*)U, guess, oT, o1, o2);
  });
}

template <typename R>
bool LaunchPoint<R>::sip(const KArgs& a, LaunchCfg lc, int K, int D, int rain, int nmembers, const long long* nvert,
    const void* U, hipStream_t s) {
  return dispatch_shape(K, D, rain, [&](auto k, auto d, auto r) {
    constexpr int K_ = decltype(k)::value, D_ = decltype(d)::value, R_ = decltype(r)::value;
    // one block per work item whatever the persistence setting (the SIP
    // kernels have no item loop)
    const dim3 grid(grid_for_items(a.nitems));
    hipLaunchKernelGGL((sip_alpha_kernel<R, K_, D_, R_>), grid, dim3(lc.threads), 0, s, a, (const R*)U);
    if constexpr (K_ != 3 || D_ != 3) {   // (Q3 hexahedra: the stage kernel does the rest)
      hipLaunchKernelGGL((sip_vertex_kernel<D_>), dim3((unsigned)((a.nvert + 127) / 128)), dim3(128), 0, s, a);
      hipLaunchKernelGGL((sip_kernel<R, K_, D_, R_>), grid, dim3(lc.threads), 0, s, a, (const R*)U);
    }
  });
}

template <typename R>
bool LaunchPoint<R>::sponge_vjp(const KArgs& a, LaunchCfg lc, int K, int D, int rain, const void* W, void* Wp,
    hipStream_t s) {
  return dispatch_shape(K, D, rain, [&](auto k, auto d, auto r) {
    constexpr int K_ = decltype(k)::value, D_ = decltype(d)::value, R_ = decltype(r)::value;
    hipLaunchKernelGGL((sponge_vjp_kernel<R, K_, D_, R_>), dim3(lc.grid), dim3(lc.threads), 0, s, a,
                       (const R*)W, (R*)Wp);
  });
}

template <typename R>
bool LaunchPoint<R>::mass(const KArgs& a, LaunchCfg lc, int K, int D, int rain, int item0, int nitems,
    const void* U, double* partial, hipStream_t s) {
  return dispatch_shape(K, D, rain, [&](auto k, auto d, auto r) {
    constexpr int K_ = decltype(k)::value, D_ = decltype(d)::value, R_ = decltype(r)::value;
    hipLaunchKernelGGL((mass_kernel<R, K_, D_, R_>), dim3(nitems), dim3(lc.threads), 0, s, a, item0,
                       (const R*)U, partial);
  });
}

template <typename R>
bool LaunchStage<R>::rhs(const KArgs& a, const KArgs* a_dev, LaunchCfg lc, int K, int D, int rain, int mode, const void* U,
    const double* auxT, const double* auxS, void* out, const void* U0,
    const double* dt, double c0, double c1, double c2, double* oT, double* oS,
    int flags, hipStream_t s) {
  return dispatch_shape(K, D, rain, [&](auto k, auto d, auto r) {
    constexpr int K_ = decltype(k)::value, D_ = decltype(d)::value, R_ = decltype(r)::value;
    dim3 grid(lc.grid), block(lc.threads);
    // (the threads beyond the nodes take face tasks)
    block = dim3(block_kernel_threads(K_, D_, lc.threads));
#define DGM_RHS(KER, M)                                                                           \
hipLaunchKernelGGL((KER<R, K_, D_, R_, M>), grid, block, 0, s, a, (const R*)U, auxT, auxS,       \
                   (R*)out, (const R*)U0, dt, c0, c1, c2, oT, oS, flags)
    // the persistent (looping) variant only when the grid is smaller than the items
    const bool persist = (int)grid.x < grid_for_items(a.nitems);
    if constexpr (K_ == 3 && D_ == 3) {
      // Q3 hexahedra: one block per brick whatever the launch geometry of the
      // other kernels
      grid = dim3(grid_for_items(a.nbricks));
      dispatch_brick(a, [&](auto bx, auto by) {
        constexpr int BX = decltype(bx)::value, BY = decltype(by)::value;
#define DGM_Q3(M, SIP)                                                                              \
  hipLaunchKernelGGL((rhs_q3_kernel<R, R_, M, SIP, BX, BY>), grid, dim3(64 * BX * BY), 0, s, a,      \
                     (const R*)U, auxT, auxS, (R*)out, (const R*)U0, dt, c0, c1, c2, oT, oS, flags)
        if (flags & kSip) {
          if (mode == 0) DGM_Q3(0, 1);
          else DGM_Q3(2, 1);
        } else {
          if (mode == 0) DGM_Q3(0, 0);
          else DGM_Q3(2, 0);
        }
      });
#undef DGM_Q3
    } else if (mode != 2 || !persist) {
      // rhs_kernel takes one work item per block: the full grid
      grid = dim3(grid_for_items(a.nitems));
      if (mode == 0) DGM_RHS(rhs_kernel, 0);
      else DGM_RHS(rhs_kernel, 2);
    } else
      hipLaunchKernelGGL((rhs_kernel_persistent<R, K_, D_, R_, 2>), grid, block, 0, s, a, a_dev, (const R*)U,
                         auxT, auxS, (R*)out, (const R*)U0, dt, c0, c1, c2, oT, oS, flags);
#undef DGM_RHS
  });
}

template <typename R>
bool LaunchGauss<R>::rhs_gauss(const KArgs& a, LaunchCfg lc, int K, int D, int rain, int mode, const void* U,
    const double* auxT, const double* auxS, void* out, const void* U0, const double* dt,
    double c0, double c1, double c2, double* oT, double* oS, int flags, hipStream_t s) {
  return dispatch_shape(K, D, rain, [&](auto k, auto d, auto r) {
    constexpr int K_ = decltype(k)::value, D_ = decltype(d)::value, R_ = decltype(r)::value;
    const dim3 grid(grid_for_items(a.nitems)), block(lc.threads);
#define DGM_RHS(M)                                                                                \
hipLaunchKernelGGL((rhs_gauss_kernel<R, K_, D_, R_, M>), grid, block, 0, s, a, (const R*)U, auxT, \
                   auxS, (R*)out, (const R*)U0, dt, c0, c1, c2, oT, oS, flags)
    if constexpr (K_ == 3 && D_ == 3) {
      if (a.nbricks > 0) {
        dispatch_brick(a, [&](auto bx, auto by) {
          constexpr int BX = decltype(bx)::value, BY = decltype(by)::value;
#define DGM_GQ3(M)                                                                                    \
  hipLaunchKernelGGL((rhs_gauss_q3_kernel<R, R_, M, BX, BY>), dim3(grid_for_items(a.nbricks)),         \
                     dim3(64 * BX * BY), 0, s, a, (const R*)U, auxT, auxS, (R*)out, (const R*)U0, dt,  \
                     c0, c1, c2, oT, oS, flags)
          if (mode == 0) DGM_GQ3(0);
          else DGM_GQ3(2);
        });
#undef DGM_GQ3
        return;
      }
    }
    if (mode == 0) DGM_RHS(0);
    else DGM_RHS(2);
#undef DGM_RHS
  });
}

template <typename R>
bool LaunchGauss<R>::gauss_trace(const KArgs& a, LaunchCfg lc, int K, int D, int rain, const void* U,
    const double* auxT, const double* auxS, hipStream_t s) {
  return dispatch_shape(K, D, rain, [&](auto k, auto d, auto r) {
    constexpr int K_ = decltype(k)::value, D_ = decltype(d)::value, R_ = decltype(r)::value;
    if constexpr (K_ == 3 && D_ == 3) {
      if (a.nbricks > 0) {
        dispatch_brick(a, [&](auto bx, auto by) {
          constexpr int BX = decltype(bx)::value, BY = decltype(by)::value;
          hipLaunchKernelGGL((gauss_q3_trace_kernel<R, R_, BX, BY>), dim3(grid_for_items(a.nbricks)),
                             dim3(64 * BX * BY), 0, s, a, (const R*)U, auxT, auxS);
        });
        return;
      }
    }
    hipLaunchKernelGGL((gauss_trace_kernel<R, K_, D_, R_>), dim3(lc.grid), dim3(lc.threads), 0, s, a,
                       (const R*)U, auxT, auxS);
  });
}

template <typename R>
bool LaunchAdjoint<R>::rhs_vjp(const KArgs& a, LaunchCfg lc, int K, int D, int rain, const void* U,
    const double* auxT, const double* auxS, const void* lam, void* out,
    const void* X1, const void* X2, const double* dt, double cx1, double cx2,
    double c1, double c2, hipStream_t s) {
  return dispatch_shape(K, D, rain, [&](auto k, auto d, auto r) {
    constexpr int K_ = decltype(k)::value, D_ = decltype(d)::value, R_ = decltype(r)::value;
    hipLaunchKernelGGL((rhs_vjp_kernel<R, K_, D_, R_>), dim3(grid_for_items(a.nitems)), dim3(lc.threads), 0, s, a, (const R*)U, auxT, auxS, (const R*)lam,
                       (R*)out, (const R*)X1, (const R*)X2, dt, cx1, cx2, c1, c2);
  });
}

template <typename R>
bool LaunchAdjoint<R>::split_vjp(const KArgs& a, LaunchCfg lc, int K, int D, int rain, const void* U,
    const double* auxT, const double* auxS, const double* Tb, const double* rvb,
    const double* rcb, void* out, hipStream_t s) {
  return dispatch_shape(K, D, rain, [&](auto k, auto d, auto r) {
    constexpr int K_ = decltype(k)::value, D_ = decltype(d)::value, R_ = decltype(r)::value;
    hipLaunchKernelGGL((split_vjp_kernel<R, K_, D_, R_>), dim3(grid_for_items(a.nitems)), dim3(lc.threads), 0, s, a, (const R*)U, auxT, auxS, Tb, rvb, rcb,
                       (R*)out);
  });
}

}  // namespace dgm
