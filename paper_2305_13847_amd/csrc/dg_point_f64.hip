// The split, diffusion, mass and sponge kernels in FP64.
#include "dg_launch_impl.h"

namespace dgm {
template struct LaunchPoint<double>;
}
