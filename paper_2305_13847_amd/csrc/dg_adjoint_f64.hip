// The adjoint kernels in FP64.
#include "dg_launch_impl.h"

namespace dgm {
template struct LaunchAdjoint<double>;
}
