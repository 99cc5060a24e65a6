// Instances of the matrix-core update: in-place step, 33 to 64 particles.
#define SVGD_UPDATE_INSTANCES
#include "update_launch.hpp"

template void svgd::launch_update_high<false, false>(const svgd::UpdateCall &);
