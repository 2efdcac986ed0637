// quad.hpp -- 16-byte accesses of 4 floats.  Clang C++ besides the function
// qualifiers, so that it also compiles for the host.
#pragma once

namespace dsk {

typedef float f32x4 __attribute__((ext_vector_type(4)));
// the same 16 bytes at any 4-byte boundary (one instruction on gfx950).  As a
// template argument the type loses its alignment, so templates take a flag or
// the value type instead.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// ANY: at any 4-byte boundary; else p is 16-byte aligned.
template <bool NT, bool ANY = false>
__device__ __forceinline__ void store_f32x4(float *p, f32x4 v) {
    if constexpr (NT && ANY)
        __builtin_nontemporal_store((f32x4_any)v, (f32x4_any *)p);
    else if constexpr (NT)
        __builtin_nontemporal_store(v, (f32x4 *)p);
    else if constexpr (ANY)
        *(f32x4_any *)p = v;
    else
        *(f32x4 *)p = v;
}

// V (float or f32x4) at any 4-byte boundary.
template <typename V>
__device__ __forceinline__ V load_any(const float *p) {
    V v;
    __builtin_memcpy(&v, p, sizeof v);
    return v;
}

template <typename V>
__device__ __forceinline__ void store_any(float *p, V v) {
    __builtin_memcpy(p, &v, sizeof v);
}

}  // namespace dsk
