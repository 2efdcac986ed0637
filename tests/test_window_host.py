"""The vector kernels' window starts (csrc/window.hpp), compiled for the host:
over dense stacks and channels of wider frames, narrow and odd, at both
parities of the stack's address, every window that a row's clamped start gives
lies inside the readable extent, and a start that was inside already is kept."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2211_00645_amd", "csrc")

SRC = r"""
#include <cstdio>
#include <initializer_list>
#include "window.hpp"
using namespace dsk;

static long bad = 0, checked = 0;

// a: parity of the stack's first element; K: the load's alignment, E: the
// alignment kept at a stack end
template <int K, int E, int LEN>
void rows(int N, int R, int C, int FC, int c0, int a) {
    const int64_t pitch = FC, plane = (int64_t)R * FC, lo = c0, hi = (int64_t)N * plane - c0;
    for (int n = 0; n < N; ++n)
        for (int r = 0; r < R; ++r) {
            const int64_t row = n * plane + r * pitch;
            const int par = (int)((row + a) & (K - 1));
            WinRange w = row_windows<K>(C, par);
            const bool first = n == 0 && near_first(r * pitch, lo);
            const bool last = n == N - 1 && near_last(row, C, hi);
            if (first || last) w = end_windows<E, LEN>(w, row, lo, hi, par);
            for (int p = -12; p < C + 12; ++p) {
                const int off = p - ((p + par) & (K - 1)), got = clamp_start(off, w);
                const bool in = row + got >= -lo && row + got + LEN <= hi;
                const bool aligned = !(first || last) ? ((par + got) & (K - 1)) == 0
                                                      : ((par + got) & (E - 1)) == 0;
                const bool kept = off < w.lo || off > w.hi || got == off;
                ++checked;
                if (!in || !aligned || !kept) {
                    if (bad++ < 5)
                        std::printf("K%d E%d %dx%dx%d of %d at %d parity %d: plane %d row %d "
                                    "pixel %d starts at %d\n", K, E, N, R, C, FC, c0, a, n, r, p,
                                    got);
                }
            }
        }
}

int main() {
    for (int N : {1, 2, 3, 7, 70})
        for (int R : {1, 2, 3, 8, 9, 33})
            for (int C = 1; C < 20; ++C)
                for (int extra : {0, 1, 2, 5})
                    for (int c0 = 0; c0 <= extra; ++c0) {
                        const int FC = C + extra;
                        // what the vector kernels take
                        if (N * R * C < 64 || R * FC < 8) continue;
                        for (int a = 0; a < 2; ++a) {
                            rows<2, 2, 6>(N, R, C, FC, c0, a);
                            rows<2, 1, 6>(N, R, C, FC, c0, a);
                        }
                        rows<1, 1, 5>(N, R, C, FC, c0, 0);
                    }
    std::printf("checked %ld bad %ld\n", checked, bad);
    return bad != 0;
}
"""


def test_window_starts_stay_inside_the_extent(tmp_path):
    src, exe = tmp_path / "window.cpp", tmp_path / "window"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__host__=", "-D__device__=",
                    "-D__forceinline__=inline", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
    assert "bad 0" in r.stdout
