#include "batch_fused.hpp"

namespace lap {
template hipError_t launch_batch_fused_t<float>(int, int, const BatchItem*, const int*, int, int, hipStream_t);
}  // namespace lap
