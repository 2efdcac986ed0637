// Real-space (affine) deskew: the stack resampled onto a Cartesian grid of
// the sample, the alternative the paper contrasts the remap with
// ("Physical principles", remap paragraph).  Raw image n, row x, column z
// images the point X = x p, Z = z p sin(a), Y = n s_z + z p cos(a)
// (s_z the scan step).  With the output's Z on the raw column grid, voxel
// (y, x, z) at Y = Y0 + y dy lies on raw column z between images
// floor(u) and floor(u) + 1, u = (Y - z p cos(a)) / s_z, and is their linear
// interpolation (zero outside the stack).
//
// The output is several times the remap's volume and each output row
// crosses many images, so a plain gather would fetch a cache line per pixel.
// The strip kernel (k_affine_strip) keeps the images a 64-column strip needs
// in an LDS ring while a workgroup sweeps y, 4 rows of the strip at once, so
// that each voxel's weights, which depend on (y, z) only, serve four voxels.
// The one-shot kernel (k_affine, one lane per 4 output columns in output
// order) covers the geometries whose images no ring holds (grids as coarse as
// the scan, |uy| = dy / s_z of 0.9994 and more; very fine scans) and rows of
// one column.
//
// Bound: writes to HBM in this output order (a kernel of the same stores and
// nothing else: 2.70 ms on the 512x512x2048 stack, 5.4 TB/s).  Measured:
//   512x512x2048, 0.4 um, 15.6 GB: 3.24 ms, 4.81 TB/s (one wavefront per
//     4-row strip with a float ring: 3.40; one row: 4.40; one-shot: 17.4)
//   150x203x1001, 45 deg, 0.2 um, 0.85 GB: 0.198 ms, 4.3 TB/s (one-shot, the
//     only kernel that took it: 1.340)
//   512x512x2048, dy 0.38 um (0.95 images a step), 5.5 GB: 1.13 ms, 4.85 TB/s
//   200x301x777, 35 deg, 0.6 um, 1.66 GB, three outputs in turn: 0.475 ms
#include <cmath>
#include <cstdint>

#include <hip/hip_runtime.h>

#include "common.hpp"
#include "deskew.h"
#include "kernels.hpp"
#include "strip.hpp"

using namespace dsk;

namespace {

constexpr int kAffBlock = 256;

template <typename TIn>
struct AffArgs {
    const TIn *in;
    float *vol;
    int64_t ny, zgroups;  // output y count; 4-column groups per row
    int32_t N, R, C;
    double u0, uy, uz;    // u = u0 + y uy - z uz
};

// Value of image n at (x, z); zero outside the stack's images.
template <typename TIn>
__device__ __forceinline__ float img_px(const AffArgs<TIn> &a, int64_t n, int64_t x, int64_t z) {
    if (n < 0 || n >= a.N) return 0.0f;
    return (float)a.in[(n * a.R + x) * a.C + z];
}

template <typename TIn>
__device__ __forceinline__ float aff_voxel(const AffArgs<TIn> &a, double uy_part, int64_t x,
                                           int64_t z) {
    double u = __dsub_rn(uy_part, __dmul_rn((double)z, a.uz));
    // far outside the stack either way: keep the image index in range
    u = u < -1.0e15 ? -1.0e15 : (u > 1.0e15 ? 1.0e15 : u);
    const double fi = floor(u);
    const double f = __dsub_rn(u, fi);
    const int64_t n0 = (int64_t)fi;
    const float whi = (float)__dsub_rn(1.0, f), wlo = (float)f;
    const float lo = img_px(a, n0, x, z), hi = img_px(a, n0 + 1, x, z);
    return fmaf(wlo, hi, whi * lo);
}

// One lane per (y, x, 4-column group), flat in output order.  VEC: C is a
// multiple of 4 and the volume 16-byte aligned (one aligned store per
// lane); otherwise each column is stored on its own, with a bound check.
template <typename TIn, bool VEC>
__global__ __launch_bounds__(kAffBlock) void k_affine(AffArgs<TIn> a) {
    const int64_t t = (int64_t)blockIdx.x * kAffBlock + threadIdx.x;
    const int64_t per_y = (int64_t)a.R * a.zgroups;
    const int64_t y = t / per_y;
    if (y >= a.ny) return;
    const int64_t rem = t - y * per_y;
    const int64_t x = rem / a.zgroups;
    const int64_t z0 = 4 * (rem - x * a.zgroups);
    const double uy_part = __dadd_rn(a.u0, __dmul_rn((double)y, a.uy));
    float *o = a.vol + (y * a.R + x) * a.C + z0;
    if constexpr (VEC) {
        f32x4 v;
        v.x = aff_voxel(a, uy_part, x, z0);
        v.y = aff_voxel(a, uy_part, x, z0 + 1);
        v.z = aff_voxel(a, uy_part, x, z0 + 2);
        v.w = aff_voxel(a, uy_part, x, z0 + 3);
        store_f32x4<true>(o, v);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (z0 + i < a.C) store_f32<true>(o + i, aff_voxel(a, uy_part, x, z0 + i));
    }
}

// Strip kernel: a workgroup of 4 wavefronts sweeps a y range of one strip of
// kStripRows rows x kStripCols columns, kChunk y values at a time, in the
// direction in which u grows.  The images a chunk needs form a band of
// consecutive images, as wide as the strip's columns and the chunk's y values
// spread over; it lives in an LDS ring of kRing images (image n in slot n mod
// kRing) holding the raw 16-bit pixels, the strip's rows interleaved, so that
// one 8-byte LDS read returns a column of an image in all rows.
//  * A voxel's weights depend on (y, z) only: 16 lanes per y value, 4
//    adjacent columns each, compute them once, in FP64, for all kStripRows
//    rows, and write each row's 4 columns with one 16-byte store.
//  * The images the next chunk adds (at most kNewImages) are loaded into
//    registers before a chunk is computed and enter the ring after it, so
//    the loads are in flight while the chunk's voxels are written; every line
//    of the stack is read once (a ring that follows the columns' diagonal, and
//    so fits any strip width, reads each line in 3-4 chunks and was slower:
//    3.95 ms against 3.2 on the 512x512x2048 stack).
//  * Column c of the window sits in place (c mod 4) * WC / 4 + c / 4 of its
//    slot (the 16 lanes of a y value then read 128 consecutive bytes), and odd
//    slots swap neighbouring 128-byte blocks, so that two y values reading
//    neighbouring images seldom meet in the same banks.
//  * PHASE: the volume's rows start at different places of a 128-byte line.
//    A strip's 256-byte runs would then leave partial lines at both ends,
//    which cost more than anything else here (150x203x1001, 0.2 um step:
//    445 us against 216), so a run starts up to 31 columns earlier, at a line boundary;
//    the strip's rows are taken phase_rows apart, the distance at which rows
//    have one phase, and keep sharing their weights.  The window is 32
//    columns wider.
// Loads take 2 pixels at any 2-byte boundary and a row's partial groups are
// stored by column, so any column count of at least 2 and any row phase runs
// here.
constexpr int kStripBlock = 256;

// 32 KB of LDS each, 48 KB with the wider window
constexpr int strip_wg_per_cu(bool phase) { return phase ? 3 : 4; }

struct StripArgs {
    AffArgs<uint16_t> a;
    int64_t ylen;        // y values per workgroup
    int64_t strips;      // row groups * ztiles
    int32_t ztiles;
    int32_t phase_rows;  // distance of a strip's rows
};

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32_any __attribute__((aligned(2)));

template <bool PHASE, bool NT>
__global__ __launch_bounds__(kStripBlock, strip_wg_per_cu(PHASE)) void k_affine_strip(StripArgs sa) {
    constexpr int NR = kStripRows;
    constexpr int WC = strip_window(PHASE);
    constexpr int kSlot = WC * 2;                           // dwords per image
    constexpr int kPairs = WC / 2;                          // column pairs per image
    constexpr int kTasks = kNewImages * kPairs / kStripBlock;
    static_assert(kTasks * kStripBlock == kNewImages * kPairs, "whole load rounds");
    __shared__ __align__(16) uint32_t ring[kRing * kSlot];
    const AffArgs<uint16_t> &a = sa.a;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const StripPlace at = strip_of_block(blockIdx.x, sa.strips);
    const int64_t yc = at.part, st = at.strip;
    const int xi = (int)(st / sa.ztiles);
    const int S = PHASE ? sa.phase_rows : 1;
    const int x0 = xi / S * (NR * S) + xi % S;
    if (x0 >= a.R) return;
    const int zb = kStripCols * (int)(st - (int64_t)xi * sa.ztiles);
    const int wb = PHASE ? zb - 32 : zb;                    // window's first column
    const int64_t y_lo = yc * sa.ylen;
    const int64_t y_hi = y_lo + sa.ylen < a.ny ? y_lo + sa.ylen : a.ny;
    const int ny_c = (int)(y_hi - y_lo);
    const int chunks = (ny_c + kChunk - 1) / kChunk;
    const bool up = a.uy > 0.0;
    const int64_t y_first = up ? y_lo : y_hi - 1;
    const int ydir = up ? 1 : -1;
    const int64_t plane = (int64_t)a.R * a.C;
    // u of column 0 at sweep index i
    auto P = [&](int i) {
        const int64_t y = y_first + (int64_t)ydir * i;
        return __dadd_rn(a.u0, __dmul_rn((double)y, a.uy));
    };
    auto fl = [](double v) { return (int)floor(v); };
    const int we = wb + WC - 1 < a.C - 1 ? wb + WC - 1 : a.C - 1;
    const double uzb = __dmul_rn((double)(wb > 0 ? wb : 0), a.uz), uze = __dmul_rn((double)we, a.uz);
    const double uz_min = uzb < uze ? uzb : uze, uz_max = uzb < uze ? uze : uzb;
    // last image the chunk whose first sweep index is i needs
    auto top_of = [&](int i) {
        return fl(__dsub_rn(P(i + kChunk - 1 < ny_c ? i + kChunk - 1 : ny_c - 1), uz_min)) + 1;
    };

    // load tasks: (image, column pair), the pair's NR rows each
    int64_t rowo[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r)
        rowo[r] = (int64_t)(x0 + r * S < a.R ? x0 + r * S : x0) * a.C;
    auto load = [&](int n, int pr, uint32_t v[NR]) {
        // images outside the stack read image 0 or N - 1 and enter as zeros
        const int64_t nc = n < 0 ? 0 : (n >= a.N ? a.N - 1 : n);
        const int pz = wb + 2 * pr;
        const uint16_t *p = a.in + nc * plane + (pz < 0 ? 0 : (pz <= a.C - 2 ? pz : a.C - 2));
#pragma unroll
        for (int r = 0; r < NR; ++r) v[r] = *(const u32_any *)(p + rowo[r]);
    };
    auto place = [](int n, int c) {   // dword of window column c of image n
        return (n & (kRing - 1)) * kSlot + 2 * (((c & 3) * (WC / 4) + (c >> 2)) ^ ((n & 1) << 4));
    };
    auto put = [&](int n, int pr, const uint32_t v[NR]) {
        const bool ok = n >= 0 && n < a.N, last_odd = wb + 2 * pr == a.C - 1;
        uint32_t w[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) w[r] = !ok ? 0u : (last_odd ? v[r] >> 16 : v[r]);
        *(u32x2 *)(ring + place(n, 2 * pr)) =
            u32x2{(w[0] & 0xffffu) | (w[1] << 16), (w[2] & 0xffffu) | (w[3] << 16)};
        *(u32x2 *)(ring + place(n, 2 * pr + 1)) =
            u32x2{(w[0] >> 16) | (w[1] & 0xffff0000u), (w[2] >> 16) | (w[3] & 0xffff0000u)};
    };

    // the first chunk's band
    int have = top_of(0);
    const int lo0 = fl(__dsub_rn(P(0), uz_max));
    for (int id = tid; id < (have - lo0 + 1) * kPairs; id += 2 * kStripBlock) {
        const int id1 = id + kStripBlock;
        const int n0 = lo0 + id / kPairs, n1 = lo0 + id1 / kPairs;
        uint32_t v0[NR], v1[NR];
        load(n0, id % kPairs, v0);
        load(n1, id1 % kPairs, v1);
        put(n0, id % kPairs, v0);
        if (n1 <= have) put(n1, id1 % kPairs, v1);
    }
    __syncthreads();

    // this lane's y within a step and its first column (less the row's phase)
    const int yq = tid >> 4;
    const int zl = zb + 4 * (lane & 15);
    double uzq[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) uzq[k] = __dmul_rn((double)(zl + k), a.uz);
    const int64_t row0 = (y_first + (int64_t)ydir * yq) * a.R + x0;
    float *out = a.vol + row0 * a.C + zl;
    const int64_t ostep = (int64_t)ydir * kChunk * plane;
    // columns between the line boundary before the row's start and that start
    int ph = 0, phstep = 0;
    if constexpr (PHASE) {
        ph = (int)(((uintptr_t)a.vol >> 2) + row0 * a.C) & 31;
        phstep = (int)ostep & 31;
    }
    int64_t orow[NR];
    bool rok[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        orow[r] = (int64_t)r * S * a.C;
        rok[r] = x0 + r * S < a.R;
    }

    for (int c = 0; c < chunks; ++c) {
        const int i0 = c * kChunk;
        // the images the next chunk adds
        uint32_t q[kTasks][NR];
        int top = have;
        if (c + 1 < chunks) {
            top = top_of(i0 + kChunk);
            top = top > have ? top : have;
#pragma unroll
            for (int t = 0; t < kTasks; ++t) {
                const int id = tid + t * kStripBlock, n = have + 1 + id / kPairs;
                load(n <= top ? n : top, id % kPairs, q[t]);
            }
        }
        {
            const int i = i0 + yq;
            const double p = P(i);
            const int zq = zl - ph;
            float wl[4], wh[4];
            u32x2 lo[4], hi[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double u =
                    __dsub_rn(p, PHASE ? __dmul_rn((double)(zq + k), a.uz) : uzq[k]);
                const double fi = floor(u);
                const double f = __dsub_rn(u, fi);
                const int n = (int)fi;
                // both weights rounded once from FP64
                wl[k] = (float)f;
                wh[k] = (float)__dsub_rn(1.0, f);
                lo[k] = *(const u32x2 *)(ring + place(n, zq + k - wb));
                hi[k] = *(const u32x2 *)(ring + place(n + 1, zq + k - wb));
            }
            f32x4 v[NR];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[0][k] = fmaf(wl[k], (float)(hi[k].x & 0xffffu), wh[k] * (float)(lo[k].x & 0xffffu));
                v[1][k] = fmaf(wl[k], (float)(hi[k].x >> 16), wh[k] * (float)(lo[k].x >> 16));
                v[2][k] = fmaf(wl[k], (float)(hi[k].y & 0xffffu), wh[k] * (float)(lo[k].y & 0xffffu));
                v[3][k] = fmaf(wl[k], (float)(hi[k].y >> 16), wh[k] * (float)(lo[k].y >> 16));
            }
            if (i < ny_c) {
                float *o = out - ph;
                if (zq >= 0 && zq + 4 <= a.C) {
#pragma unroll
                    for (int r = 0; r < NR; ++r)
                        if (rok[r]) store_f32x4<NT, true>(o + orow[r], v[r]);
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        if (zq + k < 0 || zq + k >= a.C) continue;
#pragma unroll
                        for (int r = 0; r < NR; ++r)
                            if (rok[r]) store_f32<false>(o + orow[r] + k, v[r][k]);
                    }
                }
            }
            out += ostep;
            ph = (ph + phstep) & 31;
        }
        if (c + 1 < chunks) {
            __syncthreads();
#pragma unroll
            for (int t = 0; t < kTasks; ++t) {
                const int id = tid + t * kStripBlock, n = have + 1 + id / kPairs;
                if (n <= top) put(n, id % kPairs, q[t]);
            }
            have = top;
            __syncthreads();
        }
    }
}

// y values per workgroup.  Workgroups drift apart in y as they sweep, which
// scatters the writes, so where the last-level cache holds the stack the y
// range is cut into parts of at most part_y values (strip_part; every part loads
// its first band anew); from HBM the bands cost more than the drift, and a larger
// stack is swept whole (512x512x2048, 1.07 GB: 3.23 ms, in parts of 256 3.62).
// With fewer than 4 rounds of resident workgroups the range is cut further, into
// the count of parts that fills the rounds best; a part costs its y values and
// about 24 more.
constexpr int64_t kCachedStack = 300000000;

int64_t strip_ylen(int64_t strips, int64_t ny, int wg_per_cu, int64_t stack_bytes,
                   int64_t part_y) {
    const int64_t resident = (int64_t)wg_per_cu * device_cus();
    const int64_t first = stack_bytes <= kCachedStack ? (ny + part_y - 1) / part_y : 1;
    int64_t best = first;
    if (strips * first >= 4 * resident) return first == 1 ? ny : part_y;
    double cost = 1e300;
    for (int64_t parts = first;
         parts < first + 32 && (parts == first || ny / parts >= 2 * kChunk); ++parts) {
        const double len = (double)((ny + parts - 1) / parts);
        const double rounds = (double)((strips * parts + resident - 1) / resident);
        const double c = rounds * (len + 24.0);
        if (c < 0.97 * cost) {
            cost = c;
            best = parts;
        }
    }
    const int64_t len = (ny + best - 1) / best;
    return (len + kChunk - 1) / kChunk * kChunk;
}

bool geom_ok(dsk_geom g) {
    return std::isfinite(g.angle_deg) && std::isfinite(g.step_um) && std::isfinite(g.pixel_um) &&
           g.pixel_um > 0.0 && g.step_um != 0.0;
}

}  // namespace

extern "C" int dsk_affine_plan(dsk_dims d, dsk_geom g, double dy_um, double *y0_um,
                               int64_t *ny) {
    if (!dims_ok(d) || !geom_ok(g) || !std::isfinite(dy_um) || !(dy_um > 0.0)) return DSK_EINVAL;
    const double pi = 3.14159265358979323846;
    const double pc = g.pixel_um * std::cos(g.angle_deg * pi / 180.0);
    const double c[4] = {0.0, (double)(d.planes - 1) * g.step_um, (double)(d.cols - 1) * pc,
                         (double)(d.planes - 1) * g.step_um + (double)(d.cols - 1) * pc};
    double lo = c[0], hi = c[0];
    for (int k = 1; k < 4; ++k) {
        lo = c[k] < lo ? c[k] : lo;
        hi = c[k] > hi ? c[k] : hi;
    }
    const double n = std::floor((hi - lo) / dy_um) + 1.0;
    if (!(n >= 1.0) || n >= 1.0e15) return DSK_ESHAPE;
    if (y0_um) *y0_um = lo;
    if (ny) *ny = (int64_t)n;
    return DSK_OK;
}

extern "C" int dsk_affine_u16(const uint16_t *in, dsk_dims d, dsk_geom g, double dy_um,
                              double y0_um, int64_t ny, float *vol, hipStream_t stream) {
    if (!in || !vol || !dims_ok(d) || !geom_ok(g) || !std::isfinite(dy_um) || !(dy_um > 0.0) ||
        !std::isfinite(y0_um) || ny <= 0)
        return DSK_EINVAL;
    const double pi = 3.14159265358979323846;
    const double pc = g.pixel_um * std::cos(g.angle_deg * pi / 180.0);
    AffArgs<uint16_t> a{in, vol, ny, (d.cols + 3) / 4, d.planes, d.rows, d.cols,
                        y0_um / g.step_um, dy_um / g.step_um, pc / g.step_um};
    const int64_t threads = ny * (int64_t)d.rows * a.zgroups;
    if (threads / kAffBlock >= kMaxI32) return DSK_ESHAPE;
    const dim3 grid((unsigned)((threads + kAffBlock - 1) / kAffBlock));
    // The strip kernel takes floors of u as ints: every u of the grid
    // (u0 + y uy - z uz over the whole output) must stay within +-1e9.
    const double ue[4] = {a.u0, a.u0 + (double)(ny - 1) * a.uy, a.u0 - (double)(d.cols - 1) * a.uz,
                          a.u0 + (double)(ny - 1) * a.uy - (double)(d.cols - 1) * a.uz};
    bool u_ok = true;
    for (double v : ue) u_ok = u_ok && std::fabs(v) < 1.0e9;
    auto fits = [&](bool phase) { return strip_fits(a.uy, a.uz, phase); };
    const StripStores stores =
        strip_stores(4 * ny * d.rows * (int64_t)d.cols,
                     ((uintptr_t)vol & 127) == 0 && d.cols % 32 == 0, fits(true));
    const bool phase = stores == StripStores::kPhase;
    if (u_ok && fits(phase) && d.cols >= 2 && ny < (int64_t(1) << 30) && ((uintptr_t)in & 1) == 0 &&
        ((uintptr_t)vol & 3) == 0) {
        int s = 1;   // rows s apart start at one place of a 128-byte line
        while (phase && (int64_t)s * d.cols % 32 != 0) s *= 2;
        const int64_t plane_px = (int64_t)d.rows * d.cols;
        const int32_t ztiles = (d.cols + (phase ? 31 : 0) + kStripCols - 1) / kStripCols;
        const int64_t per_class = ((int64_t)d.rows + s - 1) / s;
        const int64_t strips = s * ((per_class + kStripRows - 1) / kStripRows) * ztiles;
        const int64_t stack_bytes = 2 * (int64_t)d.planes * plane_px;
        const int64_t ylen = strip_ylen(strips, ny, strip_wg_per_cu(phase), stack_bytes,
                                        strip_part(stores, stack_bytes, a.uy, a.uz));
        const int64_t blocks = strips * ((ny + ylen - 1) / ylen);
        if (blocks < kMaxI32) {
            const StripArgs sa{a, ylen, strips, ztiles, s};
            auto go = [&](auto kern) {
                hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kStripBlock), 0, stream, sa);
            };
            if (phase)
                go(k_affine_strip<true, true>);
            else if (stores == StripStores::kLines)
                go(k_affine_strip<false, true>);
            else
                go(k_affine_strip<false, false>);
            return hip_status(hipGetLastError());
        }
    }
    const bool vec = d.cols % 4 == 0 && ((uintptr_t)vol & 15) == 0;
    if (vec)
        hipLaunchKernelGGL((k_affine<uint16_t, true>), grid, dim3(kAffBlock), 0, stream, a);
    else
        hipLaunchKernelGGL((k_affine<uint16_t, false>), grid, dim3(kAffBlock), 0, stream, a);
    return hip_status(hipGetLastError());
}
