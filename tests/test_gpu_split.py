"""The split kernel (frames of few tiles in the library's default shape): step
and chunk remainders, planes at the stack's ends, padding, and every set of
outputs; bitwise the scalar kernel (2 columns per thread)."""
import numpy as np
import pytest
import torch

import paper_2211_00645_amd as dsk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SCALAR = dict(block=64, per_thread=2, unroll=1)


@pytest.mark.parametrize("dtype", ["u16", "f32"])
@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 16, 23, 24, 31, 33, 64, 65, 129])
def test_planes(n, dtype):
    g = torch.Generator().manual_seed(n)
    for shape, shift in (((n, 3, 65), 1.7), ((n, 2, 261), -0.6), ((n, 1, 8), 9.3)):
        st = torch.randint(0, 65536, shape, generator=g, dtype=torch.int32).to(DEV)
        # float32: negative values too, so that padding's zeros are a maximum
        st = st.to(torch.uint16) if dtype == "u16" else st.float() * 0.61 - 20000.0
        offs = np.arange(n) * shift + np.random.default_rng(n).normal(0, 0.7, n)
        ref = dsk.deskew(st, offsets=offs, tune=SCALAR)
        for want in (("vol", "psum", "pmax"), ("vol",), ("psum",), ("pmax",), ("vol", "pmax"),
                     ("psum", "pmax")):
            out = dsk.deskew(st, offsets=offs, **{k: k in want for k in ("vol", "psum", "pmax")})
            torch.cuda.synchronize()
            for k in want:
                assert torch.equal(out[k], ref[k]), (shape, want, k)


def test_channel_of_a_frame():
    """Rows of a wider frame: the readable extent ends inside the frame."""
    frames = torch.randint(0, 65536, (26, 5, 150), dtype=torch.int32).to(torch.uint16).to(DEV)
    for c0 in (0, 1, 73):
        got = dsk.deskew_channels(frames, (c0,), 77, 35.0, 0.4, 0.115)[0]
        ref = dsk.deskew(frames[:, :, c0:c0 + 77].contiguous(), 35.0, 0.4, 0.115, tune=SCALAR)
        torch.cuda.synchronize()
        for k in ("vol", "psum", "pmax"):
            assert torch.equal(got[k], ref[k]), (c0, k)
