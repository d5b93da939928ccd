#include "fused_launch.hpp"

namespace lap {
template hipError_t launch_fused_v<double, 2>(const SweepArgs<double>&, int, hipStream_t);
}  // namespace lap
