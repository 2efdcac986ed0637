// split.hip -- launches of the split kernel (frames of few tiles) and of the
// row kernel (projections whose tiles meet few planes), in a translation unit
// of their own.
#include <hip/hip_runtime.h>

#include "common.hpp"
#include "kernels.hpp"

namespace dsk {

namespace {

template <typename TIn, int U>
hipError_t launch_planes(const FwdArgs<TIn> &a, int64_t tiles, hipStream_t s) {
    const dim3 grid((unsigned)(tiles * a.R)), block(kSplitBlock);
    if (a.vol)
        hipLaunchKernelGGL((k_forward_split<TIn, U, true>), grid, block, 0, s, a, (int)tiles);
    else
        hipLaunchKernelGGL((k_forward_split<TIn, U, false>), grid, block, 0, s, a, (int)tiles);
    return hipGetLastError();
}

// Planes a wavefront takes per step: 4, and 2 where that leaves wavefronts
// idle (22x128x64 uint16 with a volume 7.1 us with 4, 5.9 with 2;
// 302x64x128 47.6 and 50.9; 8 gain nothing).
template <typename TIn>
hipError_t launch(const FwdArgs<TIn> &a, int64_t tiles, hipStream_t s) {
    return a.N < 24 ? launch_planes<TIn, 2>(a, tiles, s) : launch_planes<TIn, 4>(a, tiles, s);
}

template <typename TIn>
hipError_t project(const FwdArgs<TIn> &a, hipStream_t s) {
    constexpr int64_t cols = 256 / kProjectRows;
    const int64_t tiles = (a.W + cols - 1) / cols;
    const int64_t groups = ((int64_t)a.R + kProjectRows - 1) / kProjectRows;
    hipLaunchKernelGGL(k_project_rows<TIn>, dim3((unsigned)(tiles * groups)), dim3(64), 0, s, a,
                       (int)tiles, (int)groups);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_project_rows(const FwdArgs<uint16_t> &a, hipStream_t s) { return project(a, s); }

hipError_t launch_project_rows(const FwdArgs<float> &a, hipStream_t s) { return project(a, s); }

hipError_t launch_split(const FwdArgs<uint16_t> &a, int64_t tiles, hipStream_t s) {
    return launch(a, tiles, s);
}

hipError_t launch_split(const FwdArgs<float> &a, int64_t tiles, hipStream_t s) {
    return launch(a, tiles, s);
}

#if DSK_CHECK_BOUNDS
int split_bounds_violations(unsigned long long *count, bool reset) {
    return read_bounds_violations(count, reset);
}
#endif

}  // namespace dsk
