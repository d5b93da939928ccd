// Dispatch of the fused streaming passes of one grid by columns per lane
// (kernels: fused_launch.hpp).
#include "lap_kernels.hpp"

namespace lap {

template <typename T, int V>
hipError_t launch_fused_v(const SweepArgs<T>& a, int flags, hipStream_t s);

template <typename T>
hipError_t launch_fused(const SweepArgs<T>& a, int flags, hipStream_t s) {
    const int need = ((flags & SW_FOUR) ? 8 : (flags & SW_TWO) ? 4 : 2) + ((flags & (SW_RESTRICT | SW_DEF)) ? 2 : 0);
    // the halo must cover every fused stage, in whole lanes
    if (a.tl.H < need || a.tl.H % a.tl.V != 0) return hipErrorInvalidValue;
    if (!fused_arrays(flags, a.uin, a.uout, a.f, a.ec, a.bc, a.partials, a.psi_in, a.psi_out, a.rhs_out))
        return hipErrorInvalidValue;
    switch (a.tl.V) {
        case 1: return launch_fused_v<T, 1>(a, flags, s);
        case 2: return launch_fused_v<T, 2>(a, flags, s);
        case 4: return launch_fused_v<T, 4>(a, flags, s);
        default: return hipErrorInvalidValue;
    }
}
template hipError_t launch_fused<double>(const SweepArgs<double>&, int, hipStream_t);
template hipError_t launch_fused<float>(const SweepArgs<float>&, int, hipStream_t);

}  // namespace lap
