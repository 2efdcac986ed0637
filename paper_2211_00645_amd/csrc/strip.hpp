// strip.hpp -- sizes of the affine strip kernel, the rule for the grids it
// takes and the order of its workgroups (affine.hip).  Plain C++ besides the
// function qualifiers, so that they can be checked without a device.
#pragma once

#include <math.h>
#include <stdint.h>

#include "xcd.hpp"

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

// How the output is written.  Whole lines (the volume on 128-byte boundaries,
// columns a multiple of 32) are streamed past the caches at any size.  Other
// rows leave partial lines at both ends of a strip's run: outputs of up to
// kCachedBytes go out in plain stores, whose partial lines the last-level cache
// joins; larger ones are streamed in runs that start at line boundaries
// (phase), or in plain stores where the ring does not hold the wider window.
// us, streamed -> plain, over three and over eight outputs in turn:
//   whole lines 40x64x256 into 345 (23 MB) 7.9 -> 8.6, 7.4 -> 8.8; 246x64x704
//     (215 MB) 48.1 -> 62.4; 200x100x512 (228 MB) 47.0 -> 54.9 (over one output
//     again and again 46.9 -> 39.5)
//   other rows 28x667x135 (73 MB) 34.3 -> 19.5, 34.4 -> 30.2; 200x64x333 (82 MB)
//     37.4 -> 21.1, 37.4 -> 35.6; 200x120x420 (209 MB) 50.0 -> 76.0, 49.1 -> 75.7;
//     200x99x510 (224 MB) 61.2 -> 88.5 (one output 63.0 -> 49.3)
enum class StripStores { kPlain, kLines, kPhase };

constexpr int64_t kCachedBytes = 100000000;

inline StripStores strip_stores(int64_t out_bytes, bool whole_lines, bool phase_fits) {
    if (whole_lines) return StripStores::kLines;
    return out_bytes > kCachedBytes && phase_fits ? StripStores::kPhase : StripStores::kPlain;
}

// y values of a part, where the y range is cut (affine.hip).  Parts go out in
// order, so short ones keep the planes written at a time together; each loads
// its band of images anew.  us over three outputs in turn, 256 / 64 / 32 y
// values, and the kernel before this one:
//   whole lines, stacks up to kShortPartStack: 161x64x960 (20 MB into 357) 70.4 /
//     68.3 / 57.9, before 67.2; 120x96x800 (18 MB) 67.1 / 64.2 / 55.9, 64.7;
//     100x256x512 (26 MB) 82.5 / 81.9 / 68.5, 83.6; 70x512x448 (32 MB) 138.8 / 136.6
//     / 137.4, 138.6; 200x128x1024 (52 MB) 165 / 164 / 140, 172; 120x960x256 (59 MB
//     into 897) 177 / 174 / 154, 166; 470x153x448 (64 MB) 152 / 144 / 141, 165
//   larger: 127x832x384 (81 MB) 230 / 230 / 234, 276; 363x320x448 (104 MB) 300 / 319
//     / 360, 425; 376x320x512 (123 MB) 192 / 204 / 245, 271; 100x512x1024 (105 MB)
//     520 / 483 / 544, 573; 60x1024x1024 (126 MB) 855 / 796 / 865, 953; 256x512x1024
//     (268 MB) 782 / 784 / 878, 900
//   wide bands: 200x128x512 at 0.15 um (55 images) 37.5 / 32.6 / 38.8, 119
//   runs at line boundaries (wider windows, 256 / 64): 200x301x777 479 / 514,
//     150x203x1001 133 / 147
//   plain stores: equal (200x64x333 22.9 / 23.7, 28x667x135 19.6 / 19.4)
constexpr int64_t kShortPartStack = 70000000;
constexpr double kShortPartBand = 24.0;

inline int64_t strip_part(StripStores stores, int64_t stack_bytes, double uy, double uz) {
    if (stores != StripStores::kLines) return 256;
    const double band = (strip_window(false) - 1) * fabs(uz) + kChunk * fabs(uy) + 3.0;
    return stack_bytes <= kShortPartStack && band <= kShortPartBand ? 32 : 64;
}

// Part of the y range and strip of workgroup b.  The parts go out one after
// another, so that the chip writes neighbouring planes at any time; within a
// part each XCD has a contiguous range of strips, neighbours of a row, whose
// shared lines its L2 joins.  One range per XCD over all parts had the 8 XCDs
// write 8 parts at once: us over three outputs in turn, so -> now,
// 256x256x1000 (1.7 GB, 7 parts) 494 -> 433, 256x512x1024 877 -> 782,
// 200x301x777 522 -> 479, 70x512x448 into 743 (0.7 GB) 140.6 -> 138.2,
// 300x40x1024 (0.3 GB) 65.1 -> 60.5; without the XCDs' ranges 424, 827, 458,
// 137.3 and 60.0.
struct StripPlace {
    int64_t part, strip;
};

__host__ __device__ __forceinline__ StripPlace strip_of_block(int64_t b, int64_t strips) {
    const int64_t part = b / strips;
    return StripPlace{part, xcd_remap(b - part * strips, strips)};
}

}  // namespace dsk
