// Instances of the matrix-core update: update direction, 33 to 64 particles.
#define SVGD_UPDATE_INSTANCES
#include "update_launch.hpp"

template void svgd::launch_update_high<true, false>(const svgd::UpdateCall &);
