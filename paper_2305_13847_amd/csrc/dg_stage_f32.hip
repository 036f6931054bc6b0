// The Lobatto right-hand side and stage kernels in FP32 bulk.
#include "dg_launch_impl.h"

namespace dgm {
template struct LaunchStage<float>;
}
