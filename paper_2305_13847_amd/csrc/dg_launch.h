// Host-side launchers: declarations.  They map runtime (order, dimension,
// rain) to the kernel instantiations; dg_launch_impl.h defines them, and each
// group of kernels is instantiated per precision in a translation unit of its
// own (dg_stage_f32.hip, ...), so the host code that includes this header
// compiles no kernel.
#pragma once
#include "dg_kernels.h"

namespace dgm {

inline int elems_per_block(int K, int D, bool fp64) {
  const int np = (D == 2) ? (K + 1) * (K + 1) : (K + 1) * (K + 1) * (K + 1);
  const int bt = fp64 ? block_threads<double>() : block_threads<float>();
  return bt / np > 0 ? bt / np : 1;
}

// Launch geometry of a handle: threads per block (EPB elements) and grid size.
struct LaunchCfg {
  int threads;
  int grid;
};

template <typename R>
struct LaunchPoint {
  // API != 0: write T, rho_v, rho_c; otherwise T and rho_vs(T)
  static bool split(const KArgs& a, LaunchCfg lc, int K, int D, int rain, int item0, int nitems,
                    const void* U, const double* guess, double* oT, double* o1, double* o2, int api,
                    hipStream_t s);
  // artificial diffusion: alpha_K, vertex means (all members), tendency (Q3
  // hexahedra: alpha_K only, the stage kernel does the rest)
  static bool sip(const KArgs& a, LaunchCfg lc, int K, int D, int rain, int nmembers, const long long* nvert,
                  const void* U, hipStream_t s);
  static bool sponge_vjp(const KArgs& a, LaunchCfg lc, int K, int D, int rain, const void* W, void* Wp,
                         hipStream_t s);
  static bool mass(const KArgs& a, LaunchCfg lc, int K, int D, int rain, int item0, int nitems,
                   const void* U, double* partial, hipStream_t s);
};

template <typename R>
struct LaunchStage {
  // mode 0: out = dU/dt; mode 2: out = c0 U0 + c1 U + c2 dt dU/dt and the split of out into (oT, oS)
  static bool rhs(const KArgs& a, const KArgs* a_dev, LaunchCfg lc, int K, int D, int rain, int mode, const void* U,
                  const double* auxT, const double* auxS, void* out, const void* U0,
                  const double* dt, double c0, double c1, double c2, double* oT, double* oS,
                  int flags, hipStream_t s);
};

template <typename R>
struct LaunchGauss {
  // the modes of LaunchStage::rhs on Gauss nodes: one block per work item, or per
  // brick of Q3 hexahedra, whatever the persistence setting (no item loops)
  static bool rhs_gauss(const KArgs& a, LaunchCfg lc, int K, int D, int rain, int mode, const void* U,
                        const double* auxT, const double* auxS, void* out, const void* U0, const double* dt,
                        double c0, double c1, double c2, double* oT, double* oS, int flags, hipStream_t s);
  // Gauss basis: face traces of a state and its split
  static bool gauss_trace(const KArgs& a, LaunchCfg lc, int K, int D, int rain, const void* U,
                          const double* auxT, const double* auxS, hipStream_t s);
};

template <typename R>
struct LaunchAdjoint {
  // adjoint of the right-hand side (dg_vjp.h):
  // out = cx1 X1 + cx2 X2 + c1 lam + c2 dt (d rhs/dU)^T lam   (dt = 1 if null)
  static bool rhs_vjp(const KArgs& a, LaunchCfg lc, int K, int D, int rain, const void* U,
                      const double* auxT, const double* auxS, const void* lam, void* out,
                      const void* X1, const void* X2, const double* dt, double cx1, double cx2,
                      double c1, double c2, hipStream_t s);
  static bool split_vjp(const KArgs& a, LaunchCfg lc, int K, int D, int rain, const void* U,
                        const double* auxT, const double* auxS, const double* Tb, const double* rvb,
                        const double* rcb, void* out, hipStream_t s);
};

template <typename R>
struct Launch : LaunchPoint<R>, LaunchStage<R>, LaunchGauss<R>, LaunchAdjoint<R> {};

}  // namespace dgm
