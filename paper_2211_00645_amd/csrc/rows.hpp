// rows.hpp -- the rule for the projections that go to the row kernel
// (k_project_rows: 64 columns of 4 rows a wavefront).  Plain C++, so that it can
// be checked without a device.
#pragma once

#include <stdint.h>

namespace dsk {

// Stacks of up to so many bytes stay in reach of the last-level cache while a
// launch without a volume reads them (default_tune).
constexpr int64_t kSmallProjBytes = 300000000;

// The row kernel takes frames past the split kernel's where the tiles meet at
// most kFewPlanes planes, and stacks of up to kSmallProjBytes with short rows.
// What it saves are planes that reach few of a wavefront's columns: 64 columns
// meet about (C + 64) N / (W - C) planes of a uniform scan, 256 columns
// (C + 256) N / (W - C), never more than N.  Stacks over kRowsAnyBytes whose
// tiles meet nearly as many planes either way (kRowsPlanes) lose.  us over three
// stacks in turn, k_forward_vec in its best shape -> row kernel:
//   few planes: 50x1304x87 into 3653 uint16 25.5 -> 18.6, 40x512x512 into 3846
//     15.7 -> 13.7, float32 15.2 -> 13.3
//   uint16, planes met 0.5-0.73 as many: 401x1209x130 90 -> 59, 256x900x200 57 ->
//     40, 512x1024x256 112 -> 104, 163x1280x448 (187 MB) 75.0 -> 61.3, 292x1216x320
//     (227 MB) 92.6 -> 83.2; 150x1000x448 (134 MB) 50.5 -> 51.9
//   as many, up to 100 MB: 78x1156x237 (43 MB) 34.5 -> 24.6, 54x995x125 17.8 -> 16.6
//   0.9 or as many, over 100 MB: 233x960x448 (200 MB) 75.3 -> 79.3, 400x900x384 (276
//     MB) 110.8 -> 131.5, 200x712x512 (146 MB) 66.5 -> 72.8, 300x600x500 82.7 -> 103.9
//   float32 rows: 401x1209x130 86 -> 77, 256x900x200 52.8 -> 52.3; 512x1024x256 146
//     -> 152, 300x900x300 79 -> 87
constexpr int64_t kFewPlanes = 16;
constexpr int32_t kShortRow16 = 512, kShortRow32 = 200;
constexpr int64_t kRowsAnyBytes = 100000000;
constexpr double kRowsPlanes = 0.85;

inline bool by_rows(int64_t planes, int64_t rows, int64_t cols, int64_t width, bool f32) {
    if ((cols + 256) * planes <= kFewPlanes * (width - cols)) return true;
    const int64_t bytes = planes * rows * cols * (f32 ? 4 : 2);
    if (cols > (f32 ? kShortRow32 : kShortRow16) || bytes > kSmallProjBytes) return false;
    if (bytes <= kRowsAnyBytes) return true;
    const double n = (double)planes, spread = (double)(width - cols);
    const double met64 = (double)(cols + 64) * n, met256 = (double)(cols + 256) * n;
    // both times spread, at most n planes
    const double most = n * (spread > 0.0 ? spread : 0.0);
    return (met64 < most ? met64 : most) < kRowsPlanes * (met256 < most ? met256 : most);
}

}  // namespace dsk
