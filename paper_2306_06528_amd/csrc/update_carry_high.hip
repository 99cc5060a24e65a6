// Instances of the matrix-core update: in-place step with carried sums, 33 to 64 particles.
#define SVGD_UPDATE_INSTANCES
#include "update_launch.hpp"

template void svgd::launch_update_high<false, true>(const svgd::UpdateCall &);
