// xcd.hpp -- workgroup ids and the chip's 8 XCDs.  Plain C++ besides the
// function qualifiers.
#pragma once

#include <stdint.h>

namespace dsk {

// Spread consecutive workgroup ids, which the dispatcher deals round-robin
// to the 8 XCDs, so that each XCD receives a contiguous range of logical
// tiles (neighbouring tiles of a row then share that XCD's L2).  A
// bijection on [0, n).
__host__ __device__ __forceinline__ int64_t xcd_remap(int64_t b, int64_t n) {
    constexpr int64_t kXcd = 8;
    const int64_t q = n / kXcd, rem = n % kXcd;
    const int64_t x = b % kXcd, i = b / kXcd;
    return x * q + (x < rem ? x : rem) + i;
}

}  // namespace dsk
