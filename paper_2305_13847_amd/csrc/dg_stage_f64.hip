// The Lobatto right-hand side and stage kernels in FP64.
#include "dg_launch_impl.h"

namespace dgm {
template struct LaunchStage<double>;
}
