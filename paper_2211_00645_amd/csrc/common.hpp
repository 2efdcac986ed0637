// common.hpp -- host-side helpers shared by the translation units of
// libdeskew.so (validation, launch-shape checks, HIP error mapping).
#pragma once

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "deskew.h"
#include "kernels.hpp"

namespace dsk {

constexpr int64_t kMaxI32 = 2147483647;

// Default forward launch shape (default_tune adapts its pace and pipeline to
// the frame): 64-thread workgroups, one 4-column group per
// lane, non-temporal stores, 2-plane pipeline (built for 8 waves per SIMD),
// paced at 5700 GB/s.  On the 512x512x2048 stack, back to back, the launch
// time follows the pace (bytes / pace + about 3 us) up to the cliff:
// 5600: 0.853 ms, 5700: 0.839, 5800: 0.824; past it the wavefronts fall
// behind the schedule, stop sleeping and drift apart (unpaced 1.01-1.06
// ms).  With each row's tiles on 128-byte boundaries of the volume that
// frame holds 5800 (0.828 ms over the timed runs) and its cliff lies past
// 5900, but other frames put it anywhere between 5000 and 6000 GB/s, so
// the default keeps a step of margin and dsk_deskew_autotune finds the
// cliff of a given frame on the device at hand.
constexpr dsk_tune kDefaultTune = {64, 4, 1, 2, 0, 5700};

// Default shape of launches without a volume (projections only, the live
// view): a 4-plane load-ahead keeps enough reads in flight (on the
// 512x512x2048 stack 0.228 ms against 0.240 for 2 planes), paced at 9000
// GB/s.  They only read; a pace above what the device reaches never holds a
// running wavefront back, it only makes the wavefronts whose plane range
// starts late (the frame's outer column tiles) wait for their turn instead
// of competing with the others at the start: 0.238 -> 0.219 ms on that
// stack.  With more tiles than resident workgroups a uniform scan's tiles go
// out in the order in which they meet the planes; of other frames the second
// round would wait out a schedule that began before it did (1-3% slower), so
// they are not paced (fwd_launch_vec), nor are small stacks (default_tune).
constexpr dsk_tune kDefaultProjTune = {64, 4, 1, 4, 0, 9000};

inline bool dims_ok(dsk_dims d) {
    return d.planes > 0 && d.rows > 0 && d.cols > 0;
}

inline bool tune_ok(const dsk_tune &t) {
    const bool b = t.block == 64 || t.block == 128 || t.block == 256;
    const bool j = t.per_thread == 1 || t.per_thread == 2 || t.per_thread == 4 ||
                   t.per_thread == 8;
    const bool u = t.unroll == 1 || t.unroll == 2 || t.unroll == 4;
    return b && j && u && (t.nt_store == 0 || t.nt_store == 1) && t.wg_per_cu >= 0 &&
           t.wg_per_cu <= 64 && t.pace_gbs >= 0 && t.pace_gbs <= 1000000;
}

// Compute units of the current device (cached per device).
int device_cus();

// Which kernel tiles a frame.  The aligned vector kernel applies when every
// row's flat volume and stack offsets keep one residue mod 4 across planes
// and the buffers are aligned (and, without a volume, when no columns are
// left over); the general vector kernel takes every other frame at least one
// group wide; the scalar kernel the rest, and shapes of fewer than 4 columns
// per thread.  Measured with a volume on 201x487x1531 uint16 (45 deg, odd in
// every side, 1.06 GB): scalar 0.641 ms, general 0.211 ms; projections only
// 0.283 -> 0.086 ms.  Aligned frames keep the aligned kernel with a volume:
// its tiles can start on 128-byte boundaries, which holds a faster pace
// (default_tune).
inline int vec_mode(const dsk_tune &t, dsk_dims d, int64_t width, const void *in, int in_is_f32,
                    const float *vol, int64_t in_plane) {
    if (t.per_thread < 4) return VEC_NONE;
    if ((int64_t)d.planes * d.rows * d.cols < 64 || in_plane < 8) return VEC_NONE;
    if (width >= (int64_t(1) << 27) || d.cols >= (1 << 27)) return VEC_NONE;
    const uintptr_t ia = in_is_f32 ? 15 : 7, im = in_is_f32 ? 3 : 1;
    if (((int64_t)d.rows * width) % 4 == 0 && in_plane % 4 == 0 && ((uintptr_t)in & ia) == 0 &&
        (vol ? ((uintptr_t)vol & 15) == 0 : width % 4 == 0))
        return VEC_ALIGNED;
    return width >= 4 && ((uintptr_t)in & im) == 0 && ((uintptr_t)vol & 3) == 0 ? VEC_GENERAL
                                                                                : VEC_NONE;
}

// Column tiles of one output row.  The aligned vector kernel tiles the row's
// whole 4-aligned groups (at most W/4 of them), the general one its columns
// in groups of 4 (the last moved back to end at the row's end); the scalar
// kernel tiles columns.
inline int64_t tiles_x(int64_t width, const dsk_tune &t, int vec) {
    const int64_t tile = (int64_t)t.block * t.per_thread;
    if (vec == VEC_ALIGNED) {
        const int64_t groups = width / 4, per = tile / 4;
        const int64_t n = (groups + per - 1) / per;
        return n > 0 ? n : 1;
    }
    return (width + tile - 1) / tile;
}

// Workgroups of the aligned vector kernel for the rows' unaligned edge
// columns (none when the width is a multiple of 4), which it runs first: one
// lane per (row, slot of 6).  The kernel receives the count.
inline int64_t edge_blocks(dsk_dims d, int64_t width, const dsk_tune &t, int vec) {
    if (vec != VEC_ALIGNED || width % 4 == 0) return 0;
    return (6 * (int64_t)d.rows + t.block - 1) / t.block;
}

template <int V>
using IC = std::integral_constant<int, V>;

// Calls f(IC<block>, IC<per_thread>, IC<unroll>, bool_constant<nt>) for a
// validated launch shape.
template <typename F>
auto dispatch_tune(const dsk_tune &t, F &&f) {
    auto with_u = [&](auto B, auto P) {
        auto with_nt = [&](auto U) {
            return t.nt_store ? f(B, P, U, std::true_type{}) : f(B, P, U, std::false_type{});
        };
        switch (t.unroll) {
        case 1: return with_nt(IC<1>{});
        case 2: return with_nt(IC<2>{});
        default: return with_nt(IC<4>{});
        }
    };
    auto with_p = [&](auto B) {
        switch (t.per_thread) {
        case 1: return with_u(B, IC<1>{});
        case 2: return with_u(B, IC<2>{});
        case 4: return with_u(B, IC<4>{});
        default: return with_u(B, IC<8>{});
        }
    };
    switch (t.block) {
    case 64: return with_p(IC<64>{});
    case 128: return with_p(IC<128>{});
    default: return with_p(IC<256>{});
    }
}

// Output width and columns stay below 2^30 so that every column index of the
// kernels (x' and x' - k, with k clamped to +-2^30) fits the index types.
inline int check_frame(dsk_dims d, int64_t origin, int64_t width) {
    if (width <= 0 || width >= (int64_t(1) << 30) || d.cols >= (1 << 30)) return DSK_ESHAPE;
    if (origin < -(int64_t(1) << 52) || origin > (int64_t(1) << 52)) return DSK_ESHAPE;
    return DSK_OK;
}

inline int hip_status(hipError_t e) { return e == hipSuccess ? DSK_OK : DSK_EHIP; }

// Input layout in elements (see FwdArgs): row pitch, plane pitch and the
// readable extent [in - lo, in + hi).
struct InLayout {
    int64_t row, plane, lo, hi;
};

inline InLayout dense_layout(dsk_dims d) {
    return InLayout{d.cols, (int64_t)d.rows * d.cols, 0, (int64_t)d.planes * d.rows * d.cols};
}

#if defined(DSK_CHECK_BOUNDS) && DSK_CHECK_BOUNDS
// Bounds-violation counts of the other translation units with checked kernels.
int batch_bounds_violations(unsigned long long *count, bool reset);
int split_bounds_violations(unsigned long long *count, bool reset);
#endif

// How a dense stack and its volume tile in the default shape: "lines" (aligned,
// on 128-byte boundaries of the volume), "aligned", "general" or "scalar".
const char *tiling_name(const void *in, int in_is_f32, dsk_dims d, const float *vol,
                        int64_t width);

// The same without a launch shape: the library's choice for the frame.
int launch_forward_default(const void *in, int in_is_f32, dsk_dims d, const InLayout &lay,
                           const double *offs, double shift, int64_t origin, float *vol,
                           float *psum, float *pmax, int64_t width, hipStream_t stream);

// The split kernel's launch (split.hip): a frame's tiles (per row) on checked
// arguments.
hipError_t launch_split(const FwdArgs<uint16_t> &a, int64_t tiles, hipStream_t s);
hipError_t launch_split(const FwdArgs<float> &a, int64_t tiles, hipStream_t s);
// The row kernel's launch for projections (split.hip), on checked arguments.
hipError_t launch_project_rows(const FwdArgs<uint16_t> &a, hipStream_t s);
hipError_t launch_project_rows(const FwdArgs<float> &a, hipStream_t s);

// Launchers (deskew.hip) used by the other translation units.
int launch_forward(const void *in, int in_is_f32, dsk_dims d, const double *offs,
                   double shift, int64_t origin, float *vol, float *psum, float *pmax,
                   int64_t width, const dsk_tune &t, hipStream_t stream);
int launch_forward_layout(const void *in, int in_is_f32, dsk_dims d, const InLayout &lay,
                          const double *offs, double shift, int64_t origin, float *vol,
                          float *psum, float *pmax, int64_t width, const dsk_tune &t,
                          hipStream_t stream);

}  // namespace dsk
