"""The projections' row kernel (4 rows x 64 columns a wavefront): rows mod 4,
columns mod 64, odd pitches, planes at the stack's ends, scans in both
directions and measured offsets; bitwise the scalar kernel (2 columns per
thread)."""
import numpy as np
import pytest
import torch

import paper_2211_00645_amd as dsk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SCALAR = dict(block=64, per_thread=2, unroll=1)


@pytest.mark.parametrize("dtype", ["u16", "f32"])
@pytest.mark.parametrize("shape,shift", [
    ((5, 801, 70), 1.3), ((2, 1002, 3), 0.4), ((9, 1003, 131), -40.7), ((70, 800, 33), 9.1),
    ((3, 900, 60), 100.0), ((130, 803, 7), 0.05), ((1, 2000, 200), 0.0),
    ((12, 770, 300), 130.0),                  # long rows, few planes a tile
])
@pytest.mark.parametrize("off", [0, 1])
def test_rows(shape, shift, dtype, off):
    n = shape[0] * shape[1] * shape[2]
    g = torch.Generator().manual_seed(1)
    flat = torch.randint(0, 65536, (n + off,), generator=g, dtype=torch.int32).to(DEV)
    flat = flat.to(torch.uint16) if dtype == "u16" else flat.float() * 0.3 - 9000.0
    st = flat[off:].view(shape)
    rng = np.random.default_rng(2)
    for offs in (np.arange(shape[0]) * shift, np.arange(shape[0]) * shift + rng.normal(0, 2, shape[0])):
        w, b = dsk.plan(shape, offsets=offs)
        kw = dict(offsets=offs, origin=b - 1, width=w + 1, vol=False)
        assert (w + 256) // 256 * shape[1] > 3 * 256      # past the split kernel
        ref = dsk.deskew(st, tune=SCALAR, **kw)
        for want in (("psum", "pmax"), ("pmax",)):
            out = dsk.deskew(st, psum="psum" in want, **kw)
            torch.cuda.synchronize()
            for k in want:
                assert torch.equal(out[k], ref[k]), (k, want)


def test_channel_of_a_frame():
    frames = torch.randint(0, 65536, (6, 903, 151), dtype=torch.int32).to(torch.uint16).to(DEV)
    for c0 in (0, 1, 74):
        got = dsk.deskew_channels(frames, (c0,), 77, 35.0, 4.0, 0.115, vol=False)[0]
        ref = dsk.deskew(frames[:, :, c0:c0 + 77].contiguous(), 35.0, 4.0, 0.115, vol=False,
                         tune=SCALAR)
        torch.cuda.synchronize()
        for k in ("psum", "pmax"):
            assert torch.equal(got[k], ref[k]), (c0, k)
