// Kernels of the fused streaming passes of one grid (see fused_tiles.hpp; one source file per element
// type and columns per lane instantiates launch_fused_v, so they compile side by side): pre-smoothing
// (one or two sweeps, from zero / with the input's residual norms) with the
// residual + full weighting of its result, post-smoothing (bilinear
// correction + two sweeps), and the mixed loop's FP32 post-smoothing of the
// finest level merged with the next FP64 defect correction.  One wavefront
// per (window, chunk) tile, blocks of four wavefronts dealt XCD-contiguously
// as in the one-sweep kernel.
#pragma once

#include "fused_tiles.hpp"

namespace lap {

// Whether a fused pass stores its rows nontemporally (past L2 and the
// Infinity Cache).  Measured on an 8193^2 solve: for the FP64 multigrid
// passes of every level it saves ~15 us per cycle on the coarser levels and
// is even on the finest (7.00 -> 6.85 ms); the FP32 passes of the mixed loop
// and the SOR passes (whose output the next pass reads at once) gain
// nothing or lose, and keep ordinary stores, as do merged batch launches of
// small grids.
template <typename T, int FL>
constexpr bool fused_nt() {
    return sizeof(T) == 8 && (FL & (SW_RESTRICT | SW_PROLONG)) != 0;
}

template <typename T, int V, int FL>
__global__ __launch_bounds__(kBlock) void k_fused(SweepArgs<T> A) {
    if (A.ctrl != nullptr && A.ctrl->done) return;
    const int tile = xcd_remap(blockIdx.x, gridDim.x) * kWavesPerBlock + wave_in_block();
    if (tile >= A.tl.ntiles) return;
    fused_tile<T, V, FL, fused_nt<T, FL>()>(A, tile, threadIdx.x & 63);
}

// The flag sets a V-cycle plan uses (SW_F added where a right-hand side exists).
#define LAP_FUSED_FLAGS(X)                                                                         \
    X(SW_TWO) X(SW_TWO | SW_F) X(SW_TWO | SW_ZERO | SW_F) X(SW_TWO | SW_NORM)                    \
    X(SW_TWO | SW_NORM | SW_F) X(SW_TWO | SW_PROLONG) X(SW_TWO | SW_PROLONG | SW_F)              \
    X(SW_TWO | SW_PROLONG | SW_ZERO | SW_F)                                                        \
    X(SW_RESTRICT) X(SW_RESTRICT | SW_F) X(SW_RESTRICT | SW_ZERO | SW_F) X(SW_RESTRICT | SW_NORM) \
    X(SW_RESTRICT | SW_NORM | SW_F) X(SW_RESTRICT | SW_TWO) X(SW_RESTRICT | SW_TWO | SW_F)       \
    X(SW_RESTRICT | SW_TWO | SW_ZERO | SW_F) X(SW_RESTRICT | SW_TWO | SW_NORM)                    \
    X(SW_RESTRICT | SW_TWO | SW_NORM | SW_F)                                                        \
    X(SW_PROBE | SW_RESTRICT | SW_TWO | SW_NORM) X(SW_PROBE | SW_RESTRICT | SW_TWO | SW_NORM | SW_F)  \
    X(SW_PROBE | SW_RESTRICT | SW_NORM) X(SW_PROBE | SW_RESTRICT | SW_NORM | SW_F)                \
    X(SW_PROBE | SW_TWO | SW_NORM) X(SW_PROBE | SW_TWO | SW_NORM | SW_F)
// FP64 only: four sweeps of red-black SOR, and a cycle's post-smoothing with
// the next one's pre-smoothing (on the norms' tiling: two columns per lane)
#define LAP_FUSED_FLAGS64(X)                                                                       \
    X(SW_FOUR) X(SW_FOUR | SW_F)                                                                   \
    X(V == 2 ? SW_FOUR | SW_PROLONG | SW_NORM | SW_RESTRICT : SW_UNUSED)                           \
    X(V == 2 ? SW_FOUR | SW_PROLONG | SW_NORM | SW_RESTRICT | SW_F : SW_UNUSED | SW_F)
// FP32 only: the mixed loop's post-smoothing + defect pass and the passes of
// a step's cycles after the first
// (post + defect only with the two columns per lane of its fixed tiling)
#define LAP_FUSED_FLAGS32(X)                                                                       \
    X(V == 2 ? SW_DEF | SW_PROLONG | SW_TWO | SW_F : SW_UNUSED) X(SW_RDIFF | SW_RESTRICT | SW_TWO | SW_F)                \
    X(SW_RDIFF | SW_RESTRICT | SW_F) X(SW_FOUR | SW_PROLONG | SW_RESTRICT | SW_RDIFF | SW_F)

template <typename T, int V>
hipError_t launch_fused_v(const SweepArgs<T>& a, int flags, hipStream_t s) {
    const dim3 grid(blocks_for(a.tl)), block(kBlock);
    switch (flags) {
#define LAP_CASE(F)                                      \
    case (F):                                            \
        if constexpr (((F) & SW_UNUSED) != 0)            \
            return hipErrorInvalidValue;                 \
        else                                             \
            k_fused<T, V, (F)><<<grid, block, 0, s>>>(a);\
        break;
        LAP_FUSED_FLAGS(LAP_CASE)
        default:
            if constexpr (sizeof(T) == 4) {
                switch (flags) {
                    LAP_FUSED_FLAGS32(LAP_CASE)
                    default: return hipErrorInvalidValue;
                }
            } else {
                switch (flags) {
                    LAP_FUSED_FLAGS64(LAP_CASE)
                    default: return hipErrorInvalidValue;
                }
            }
#undef LAP_CASE
    }
    return hipGetLastError();
}

}  // namespace lap
