// The Gauss-basis kernels in FP64.
#include "dg_launch_impl.h"

namespace dgm {
template struct LaunchGauss<double>;
}
