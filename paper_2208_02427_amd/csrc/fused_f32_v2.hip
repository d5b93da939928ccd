#include "fused_launch.hpp"

namespace lap {
template hipError_t launch_fused_v<float, 2>(const SweepArgs<float>&, int, hipStream_t);
}  // namespace lap
