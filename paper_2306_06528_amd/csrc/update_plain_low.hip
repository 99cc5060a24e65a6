// Instances of the matrix-core update: in-place step, 13 to 32 particles.
#define SVGD_UPDATE_INSTANCES
#include "update_launch.hpp"

template void svgd::launch_update_low<false, false>(const svgd::UpdateCall &);
