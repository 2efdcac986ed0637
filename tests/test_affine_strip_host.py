"""The rules of the affine strip kernel (csrc/strip.hpp), compiled for the host.
Grids: it takes scan steps up to 0.999 images per y value, and on every
grid it takes the kernel's bookkeeping -- the last image of a chunk against
that of the one before, the band against the ring -- stays within the loads of
a chunk and the ring, in 64-bit arithmetic as on the device.  Workgroups: the
parts of the y range in order, each strip of a part once, an XCD's workgroups
of a part on neighbouring strips.  Stores: whole lines streamed at any size.
Parts: the lengths measured fastest."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2211_00645_amd", "csrc")

SRC = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <initializer_list>
#include <random>
#include <vector>
#include "strip.hpp"
using namespace dsk;

int main() {
    int bad = 0;
    auto need = [&](bool ok, const char *what, double uy, double uz) {
        if (!ok && bad++ < 8) std::printf("%s: uy %.17g uz %.17g\n", what, uy, uz);
    };
    // one row of 64 columns kept 63 |uz| + 9 |uy| + 4 images of a ring of 32
    for (double uy = 0.01; uy <= 0.999; uy += 0.001)
        for (double uz : {0.0, 0.1, 0.2, (28.0 - 9.0 * uy) / 63.0})
            need(strip_fits(uy, uz, false) && strip_fits(-uy, -uz, false), "refused", uy, uz);
    need(strip_fits(0.38 / 0.4, 0.115 * 0.819152 / 0.4, true), "refused", 0.38 / 0.4, 0.0);
    need(!strip_fits(1.0, 0.0, false) && !strip_fits(-1.0, 0.1, true), "taken", 1.0, 0.0);

    std::mt19937_64 rng(3);
    auto uni = [&](double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); };
    long grids = 0;
    for (int it = 0; it < 60000; ++it) {
        const bool phase = it & 1;
        double uy = uni(0.0, 1.0), uz = uni(-0.9, 0.9);
        if (it % 3 == 0) uy = uni(0.99, 0.9995);
        if (it % 5 == 0) uy = std::floor(uy * 16.0) / 16.0;       // steps on whole images
        if (uy == 0.0 || !strip_fits(uy, uz, phase)) continue;
        ++grids;
        const double u0 = it % 7 ? uni(-600.0, 600.0) : uni(-9e8, 9e8);
        const int C = 1 + (int)uni(1, 300), WC = strip_window(phase);
        const int zb = kStripCols * (int)uni(0, (C + kStripCols - 1) / kStripCols);
        const int wb = phase ? zb - 32 : zb, we = wb + WC - 1 < C - 1 ? wb + WC - 1 : C - 1;
        const double a = (double)(wb > 0 ? wb : 0) * uz, b = (double)we * uz;
        const double lo = a < b ? a : b, hi = a < b ? b : a;
        auto P = [&](int i) { return u0 + (double)i * uy; };
        auto top = [&](int i) { return (int64_t)std::floor(P(i + kChunk - 1) - lo) + 1; };
        int64_t have = top(0);
        for (int i0 = 0; i0 < 60 * kChunk; i0 += kChunk) {
            const int64_t first = (int64_t)std::floor(P(i0) - hi);
            need(have - first + 1 <= kRing, "band", uy, uz);
            // the images of the chunk's voxels are in the ring
            need((int64_t)std::floor(P(i0 + kChunk - 1) - lo) + 1 <= have, "missing", uy, uz);
            int64_t next = top(i0 + kChunk);
            next = next > have ? next : have;
            need(next - have <= kNewImages, "loads", uy, uz);
            have = next;
        }
    }
    // whole lines are streamed at any size; other rows by the output's size
    for (int64_t bytes : {1000ll, 215000000ll, 4000000000ll})
        for (bool fits : {false, true}) {
            need(strip_stores(bytes, true, fits) == StripStores::kLines, "lines", bytes, fits);
            need((strip_stores(bytes, false, fits) == StripStores::kPhase) ==
                     (fits && bytes > 200000000), "other rows", bytes, fits);
        }
    // short parts for whole lines of small stacks that a part's band does not burden
    need(strip_part(StripStores::kLines, 20000000, 0.26, 0.22) == 32 &&
             strip_part(StripStores::kLines, 59000000, 0.17, 0.14) == 32 &&
             strip_part(StripStores::kLines, 104000000, 0.17, 0.14) == 64 &&
             strip_part(StripStores::kLines, 26000000, 0.77, 0.63) == 64 &&
             strip_part(StripStores::kPhase, 62000000, 0.65, 0.26) == 256 &&
             strip_part(StripStores::kPlain, 8000000, 0.29, 0.24) == 256,
         "part", 0.0, 0.0);
    for (int64_t strips : {1, 2, 7, 8, 9, 176, 1001, 4096})
        for (int64_t parts : {1, 2, 5}) {
            std::vector<int> seen(strips * parts, 0);
            for (int64_t b = 0; b < strips * parts; ++b) {
                const StripPlace p = strip_of_block(b, strips);
                need(p.part == b / strips, "part out of order", (double)b, (double)strips);
                need(p.strip >= 0 && p.strip < strips && !seen[p.part * strips + p.strip]++,
                     "strip", (double)b, (double)strips);
                // the next workgroup on this XCD
                if (b + 8 < (p.part + 1) * strips)
                    need(strip_of_block(b + 8, strips).strip == p.strip + 1, "neighbour",
                         (double)b, (double)strips);
            }
        }
    std::printf("grids %ld bad %d\n", grids, bad);
    return bad != 0 || grids < 10000;
}
"""


def test_strip_rule(tmp_path):
    src, exe = tmp_path / "strip.cpp", tmp_path / "strip"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-D__host__=",
                    "-D__device__=", "-D__forceinline__=inline", "-I", CSRC, str(src), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
    assert "bad 0" in r.stdout
