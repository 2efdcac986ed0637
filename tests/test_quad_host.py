"""16-byte accesses of 4 floats (csrc/quad.hpp) at every 4-byte boundary,
compiled for the host under the alignment sanitizer: the unaligned forms never
claim more alignment than the address has, and move the right bytes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2211_00645_amd", "csrc")

SRC = r"""
#include <cstdio>
#include <cstring>
#include "quad.hpp"
using namespace dsk;

template <class F>
int check(const char *what, F store) {
    alignas(16) float buf[12];
    for (int off = 0; off < 8; ++off) {
        for (int i = 0; i < 12; ++i) buf[i] = -1.0f;
        store(buf + off, f32x4{1.0f, 2.0f, 3.0f, 4.0f});
        for (int i = 0; i < 12; ++i)
            if (buf[i] != (i >= off && i < off + 4 ? (float)(i - off + 1) : -1.0f)) {
                std::printf("%s at %d\n", what, off);
                return 1;
            }
        const f32x4 v = load_any<f32x4>(buf + off);
        if (v.x != 1.0f || v.w != 4.0f || load_any<float>(buf + off + 1) != 2.0f) return 1;
    }
    return 0;
}

int main() {
    return check("store", [](float *p, f32x4 v) { store_f32x4<false, true>(p, v); }) +
           check("non-temporal store", [](float *p, f32x4 v) { store_f32x4<true, true>(p, v); }) +
           check("value", [](float *p, f32x4 v) { store_any(p, v); });
}
"""


def test_unaligned_quads(tmp_path):
    cxx = shutil.which("amdclang++") or "/opt/rocm/bin/amdclang++"
    if not os.path.exists(cxx):
        pytest.skip("no clang++")
    src, exe = tmp_path / "quad.cpp", tmp_path / "quad"
    src.write_text(SRC)
    subprocess.run([cxx, "-x", "c++", "-std=c++17", "-O1", "-fsanitize=alignment",
                    "-fno-sanitize-recover=alignment", "-fsanitize-trap=alignment",
                    "-D__device__=", "-D__forceinline__=inline", "-I", CSRC, str(src), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout)
