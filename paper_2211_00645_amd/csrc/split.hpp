// split.hpp -- the rule for the frames that go to the split kernel
// (k_forward_split: four wavefronts share a tile of 256 columns).  Plain C++, so
// that it can be checked without a device.
#pragma once

#include <stdint.h>

namespace dsk {

// The split kernel hides a chain of plane latencies that one or two tiles a SIMD
// do not, and pays with a pass through LDS and with loads in planes that miss
// the tile, which the vector kernel only fills with zeros.  So the limits are in
// tiles per compute unit, in quarters, by what the launch writes.  us over three
// stacks in turn, k_forward_vec in the default's shape -> split (tiles a unit):
//   volume and projections: 75x64x576 float32 (1.0) 20.4 -> 12.0, 302x64x128 (1.25)
//     70 -> 42, 117x73x1008 (2.0) 30.7 -> 21.3, 61x192x384 (2.25) 17.7 -> 15.8; 88x99x925
//     (2.3) 19.2 -> 19.7; 256x256x512 (5) 76 -> 103
//   the same where a tile meets under half of the planes (2 (C + 256) < W - C):
//     258x64x256 into 1276 (1.25) 43.9 -> 38.7; 413x64x128 into 2160 (2.25) 59 -> 81
//   volume alone (no sums, so no LDS and no barriers), up to kSplitPlanes: 54x177x348
//     (2.1) 16.6 -> 13.4, 128x256x512 (4) 35.6 -> 26.6; more planes: 270x128x704 (3.0)
//     68 -> 58, 505x128x384 (3.0) 155 -> 118; 253x151x781 (3.5) 59 -> 73, 437x192x320
//     (4.5) 108 -> 156, 311x288x574 (5.6) 115 -> 161
//   projections alone: 99x64x768 (1.25) 25.2 -> 16.8, 227x128x640 (3) 46.5 -> 31.6;
//     128x320x512 (5) 30.7 -> 32.1
constexpr int64_t kSplitVolume = 10, kSplitVolumeFew = 7, kSplitProjections = 12;
constexpr int64_t kSplitVolumeAlone = 24, kSplitVolumeAloneLong = 12, kSplitPlanes = 128;

inline bool by_split(int64_t planes, int64_t rows, int64_t cols, int64_t width, bool vol,
                     bool sums, int64_t cus) {
    int64_t quarters = kSplitProjections;
    if (vol && sums)
        quarters = 2 * (cols + 256) < width - cols ? kSplitVolumeFew : kSplitVolume;
    else if (vol)
        quarters = planes <= kSplitPlanes ? kSplitVolumeAlone : kSplitVolumeAloneLong;
    return 4 * ((width + 255) / 256) * rows <= quarters * cus;
}

}  // namespace dsk
