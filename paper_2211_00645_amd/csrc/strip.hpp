// strip.hpp -- sizes of the affine strip kernel and the rule for the grids it
// takes (affine.hip).  Plain C++, so that the rule can be checked without a
// device.
#pragma once

#include <math.h>

namespace dsk {

constexpr int kStripRows = 4;
constexpr int kStripCols = 64;
constexpr int kRing = 64;        // images in the LDS ring
constexpr int kNewImages = 16;   // images a chunk may add
constexpr int kChunk = 16;       // y values

// Columns of the window of images a strip keeps (phase: the strip's runs start
// at a line boundary up to 31 columns earlier).
constexpr int strip_window(bool phase) { return kStripCols + (phase ? 32 : 0); }

// Whether the ring holds what a sweep needs, the image coordinate being
// u = u0 + y uy - z uz:
//  * a chunk's last image floor(u) + 1 moves by kChunk |uy| from chunk to
//    chunk, so by at most kNewImages whole images where kChunk |uy| is at most
//    that; 0.01 is far above the rounding of u (|u| stays below 1e9).  Steps as
//    coarse as the scan (|uy| of 1 and more) go to the one-shot kernel: a chunk
//    could add one image more than its loads hold.
//  * the band of a chunk spans its columns and y values, and 3 images besides:
//    both ends' partial images and the upper neighbour.
inline bool strip_fits(double uy, double uz, bool phase) {
    const double move = kChunk * fabs(uy);
    return move + 0.01 <= kNewImages &&
           (strip_window(phase) - 1) * fabs(uz) + move + 3.0 <= kRing;
}

}  // namespace dsk
