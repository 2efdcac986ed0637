"""The rule for the split kernel (csrc/split.hpp), compiled for the host, on a
device of 256 compute units at frames measured on both sides of it: planes, rows,
columns, width, volume, sums, and which of the two kernels was the faster."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2211_00645_amd", "csrc")

FRAMES = [
    # the split kernel
    (75, 64, 576, 903, 1, 1, 1), (302, 64, 128, 1093, 1, 1, 1), (117, 73, 1008, 1554, 1, 1, 1),
    (61, 192, 384, 702, 1, 1, 1), (258, 64, 256, 1276, 1, 1, 1), (64, 128, 256, 446, 1, 1, 1),
    (54, 177, 348, 594, 1, 0, 1), (128, 256, 512, 876, 1, 0, 1), (270, 128, 704, 1343, 1, 0, 1),
    (505, 128, 384, 1418, 1, 0, 1), (99, 64, 768, 1053, 0, 1, 1), (227, 128, 640, 1289, 0, 1, 1),
    # the vector kernel
    (256, 256, 512, 1238, 1, 1, 0), (413, 64, 128, 2160, 1, 1, 0), (253, 151, 781, 1331, 1, 0, 0),
    (437, 192, 320, 1293, 1, 0, 0), (311, 288, 574, 1129, 1, 0, 0), (200, 512, 512, 1000, 1, 0, 0),
    (128, 320, 512, 876, 0, 1, 0), (512, 512, 2048, 3504, 1, 1, 0),
]


def test_measured_frames(tmp_path):
    src, exe = tmp_path / "split.cpp", tmp_path / "split"
    rows = "\n".join(f"    if (dsk::by_split({n}, {r}, {c}, {w}, {v}, {s}, 256) != {want}) "
                     f'std::printf("{n}x{r}x{c} into {w} {v}{s}\\n"), ++bad;'
                     for n, r, c, w, v, s, want in FRAMES)
    src.write_text('#include <cstdio>\n#include "split.hpp"\n'
                   f"int main() {{\n    int bad = 0;\n{rows}\n    return bad;\n}}\n")
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
