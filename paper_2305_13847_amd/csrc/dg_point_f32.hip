// The split, diffusion, mass and sponge kernels in FP32 bulk.
#include "dg_launch_impl.h"

namespace dgm {
template struct LaunchPoint<float>;
}
