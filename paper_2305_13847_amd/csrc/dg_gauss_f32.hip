// The Gauss-basis kernels in FP32 bulk.
#include "dg_launch_impl.h"

namespace dgm {
template struct LaunchGauss<float>;
}
