"""The checking build (libdeskew_bounds.so) over the paths that
test_gpu_bounds.py's shapes do not reach: projections in the row kernel, frames
and volumes off alignment in every vector shape, one-column stacks at an odd
address, channels of both, and job lists whose table travels in the launch's
arguments.  No address lies outside its buffer.  (The rolling update, the view's
stretch and the affine kernels carry no checks.)"""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2211_00645_amd", "libdeskew_bounds.so")

CHILD = r"""
import ctypes, sys
import numpy as np
import torch
sys.path.insert(0, sys.argv[1])
import paper_2211_00645_amd as dsk
from paper_2211_00645_amd import _lib as L
from paper_2211_00645_amd.batch import JobLauncher, plan_job

lib = L.lib()
cnt = ctypes.c_ulonglong(0)
assert lib.dsk_debug_bounds_violations(ctypes.byref(cnt), 1) == 1, "not a checking build"
DEV = "cuda:0"

def say(m):
    print(m, flush=True)

def stack(shape, off, dt="u16"):
    n = shape[0] * shape[1] * shape[2]
    flat = torch.randint(0, 65536, (n + off,), dtype=torch.int32, device=DEV)
    flat = flat.to(torch.uint16) if dt == "u16" else flat.float()
    return flat[off:].view(shape)

def offsets(n, s):
    return np.arange(n) * s + np.random.default_rng(n).normal(0, 0.7, n)

VECTOR = [dict(block=64, per_thread=4, unroll=2), dict(block=64, per_thread=4, unroll=4),
          dict(block=256, per_thread=8, unroll=1, pace_gbs=5000)]

# projections in the row kernel: rows mod 4, odd pitches, both ends of the stack
for shape, s in (((5, 801, 70), 1.3), ((6, 903, 77), 9.0), ((2, 1002, 3), 0.4),
                 ((9, 1003, 131), -40.7), ((3, 900, 60), 100.0), ((1, 2000, 200), 0.0),
                 ((70, 802, 1), 0.3), ((3, 1001, 1), -8.0)):
    for dt in ("u16", "f32"):
        for off in (0, 1):
            dsk.deskew(stack(shape, off, dt), offsets=offsets(shape[0], s), vol=False)
    say(f"rows {shape}")

# any alignment, one column and a few, in the default and in vector shapes
for shape, s in (((2, 33, 1), 0.3), ((70, 9, 1), 1.7), ((65, 3, 2), -0.4), ((130, 5, 3), 2.2),
                 ((9, 5, 4), 0.0), ((6, 7, 251), 1.3), ((67, 3, 255), 0.5), ((3, 33, 1021), 0.9)):
    for dt in ("u16", "f32"):
        for off in (0, 1):
            st = stack(shape, off, dt)
            offs = offsets(shape[0], s)
            w, b = dsk.plan(shape, offsets=offs)
            w = max(w, 4)
            vol = torch.empty(shape[0] * shape[1] * w + off, device=DEV)[off:]
            vol = vol.view(shape[0], shape[1], w)
            for tune in [None] + VECTOR:
                for want in ("vol", "proj"):
                    dsk.deskew(st, offsets=offs, origin=b, width=w, vol=want == "vol",
                               out={"vol": vol}, tune=tune)
            dsk.deskew(st, offsets=offs, origin=b, width=w, psum=False, pmax=False,
                       out={"vol": vol})
    say(f"general {shape}")

# channels: rows of a wider frame at both parities
for shape, cols in (((6, 903, 151), 77), ((40, 5, 75), 1), ((26, 5, 151), 77)):
    for off in (0, 1):
        frames = stack(shape, off)
        for c0 in (0, 1, shape[2] - cols):
            for vol in (True, False):
                dsk.deskew_channels(frames, (c0,), cols, 35.0, 0.4, 0.115, vol=vol)
    say(f"channel {shape}")

# job lists: the table in the arguments (up to 32 jobs) and copied
launcher = JobLauncher(max_jobs=40)
for n_jobs in (1, 9, 32, 33):
    for kind in ("vol", "proj", "mixed"):
        jobs, keep = [], []
        for i in range(n_jobs):
            st = stack((1 + 7 * i % 23, 1 + 5 * i % 19, 1 + 37 * i % 301), i % 2)
            job, out = plan_job(st, 35.0, 0.4, 0.115,
                                vol=kind == "vol" or (kind == "mixed" and i % 2 == 0))
            jobs.append(job)
            keep.append((st, out))
        launcher.launch(jobs)
        torch.cuda.synchronize()
    say(f"jobs {n_jobs}")

torch.cuda.synchronize()
assert lib.dsk_debug_bounds_violations(ctypes.byref(cnt), 0) == 1
print(f"violations {cnt.value}", flush=True)
"""


def test_no_address_outside_its_buffer():
    assert os.path.exists(LIB), ("the checking library is missing: "
                                 "python -m paper_2211_00645_amd.build --bounds")
    env = dict(os.environ, DSK_LIB=LIB)
    r = subprocess.run([sys.executable, "-u", "-c", CHILD, ROOT], env=env, cwd=ROOT,
                       capture_output=True, text=True, timeout=110)
    print(r.stdout[-4000:])
    print(r.stderr[-4000:])
    assert r.returncode == 0, "child failed"
    assert "violations 0" in r.stdout
