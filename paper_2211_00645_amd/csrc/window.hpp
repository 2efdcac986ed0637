// window.hpp -- where the vector kernels' pixel windows may start, in elements
// from the first pixel of their row.  Plain C++ besides the function
// qualifiers, so that the rules can be checked without a device.
#pragma once

#include <stdint.h>

namespace dsk {

struct WinRange {
    int lo, hi;
};

// Window starts in a row of C pixels: at most 8 elements before the row, not
// past its last pixel, and at a multiple of K elements (K = 1 or 2; par: the
// row start's residue mod K).  A window reaches at most 5 elements past the
// row.
template <int K>
__host__ __device__ __forceinline__ WinRange row_windows(int C, int par) {
    return WinRange{-8 + (par & (K - 1)), C - 1 - ((C - 1 + par) & (K - 1))};
}

// Whether a row that starts at element `row` of its stack (in plane 0, or in
// plane N - 1) lies so near the end of the readable extent [-in_lo, in_hi) that
// row_windows alone could leave it.
__host__ __device__ __forceinline__ bool near_first(int64_t row, int64_t in_lo) {
    return row - 8 < -in_lo;
}
__host__ __device__ __forceinline__ bool near_last(int64_t row, int C, int64_t in_hi) {
    return row + C + 8 > in_hi;
}

// The starts of w that keep a window of LEN elements inside the readable
// extent, at a multiple of K elements.  Where none is left (a row of one pixel
// at the very start, whose only pixel lies before the first aligned start) the
// lower end wins: it lies inside the extent, which holds at least 64 elements.
template <int K, int LEN>
__host__ __device__ __forceinline__ WinRange end_windows(WinRange w, int64_t row, int64_t in_lo,
                                                         int64_t in_hi, int par) {
    int64_t lo = -row - in_lo, hi = in_hi - LEN - row;
    lo += (par + lo) & (K - 1);
    hi -= (par + hi) & (K - 1);
    w.lo = lo > (int64_t)w.lo ? (int)lo : w.lo;
    w.hi = hi < (int64_t)w.hi ? (int)hi : w.hi;
    w.hi = w.hi < w.lo ? w.lo : w.hi;
    return w;
}

__host__ __device__ __forceinline__ int clamp_start(int off, WinRange w) {
    return off < w.lo ? w.lo : (off > w.hi ? w.hi : off);
}

}  // namespace dsk
