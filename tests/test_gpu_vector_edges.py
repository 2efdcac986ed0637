"""The vector kernel in explicit shapes with a volume, where the library's
default sends frames this small to the split kernel: tile grids on 128-byte
boundaries, planes at the stack's ends and around a chunk of 64, buffers off
alignment, and the general form as bands of rows.  Bitwise the scalar kernel
(2 columns per thread, pinned to the oracle by the forward tests)."""
import numpy as np
import pytest
import torch

import paper_2211_00645_amd as dsk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SCALAR = dict(block=64, per_thread=2, unroll=1)
VECTOR = [dict(block=64, per_thread=4, unroll=2), dict(block=64, per_thread=4, unroll=4),
          dict(block=64, per_thread=8, unroll=2, pace_gbs=5000)]
KEYS = ("vol", "psum", "pmax")


def _stack(shape, dtype, off, seed=3):
    n = shape[0] * shape[1] * shape[2]
    g = torch.Generator().manual_seed(seed)
    flat = torch.randint(0, 65536, (n + off,), generator=g, dtype=torch.int32).to(DEV)
    flat = flat.to(torch.uint16) if dtype == "u16" else flat.float() * 0.37 - 9000.0
    return flat[off:].view(shape)


def _volume(shape, lead):
    n = shape[0] * shape[1] * shape[2]
    flat = torch.full((n + lead,), float("nan"), device=DEV)
    assert flat.data_ptr() % 128 == 0
    return flat[lead:].view(shape)


@pytest.mark.parametrize("dtype", ["u16", "f32"])
@pytest.mark.parametrize("width,lead", [(1256, 0), (1272, 0), (1276, 0), (1280, 0), (1280, 4),
                                        (1112, 12), (1256, 1), (1280, 3)])
def test_tile_grids(width, lead, dtype):
    """rows * W a multiple of 32: the rows' tiles start on 128-byte boundaries
    of the volume where the shifted grids need no more tiles (1256, 1280 on a
    boundary, 1112 twelve floats after one), on plain grids otherwise, and in
    the general form where the volume is off alignment."""
    st = _stack((8, 32, 1024), dtype, 0)
    ref = dsk.deskew(st, 35.0, 0.4, 0.115, width=width, tune=SCALAR)
    for tune in VECTOR:
        vol = _volume((8, 32, width), lead)
        out = dsk.deskew(st, 35.0, 0.4, 0.115, width=width, out={"vol": vol}, tune=tune)
        torch.cuda.synchronize()
        for k in KEYS:
            assert torch.equal(out[k], ref[k]), (tune, k)


@pytest.mark.parametrize("dtype", ["u16", "f32"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129])
@pytest.mark.parametrize("r,c,off", [(4, 64, 0), (4, 96, 0), (3, 65, 0), (5, 61, 1), (9, 8, 1)])
def test_stack_ends(n, r, c, off, dtype):
    """One plane that holds the first and the last rows, chunks of 1, 63 and 64
    planes; the aligned and the general form."""
    st = _stack((n, r, c), dtype, off)
    rng = np.random.default_rng(n)
    for offs in (np.arange(n) * 2.718281828, np.arange(n) * -1.4142135,
                 np.arange(n) * 0.3 + rng.normal(0, 1, n)):
        ref = dsk.deskew(st, offsets=offs, tune=SCALAR)
        for tune in VECTOR:
            out = dsk.deskew(st, offsets=offs, tune=tune,
                             out={"vol": _volume(tuple(ref["vol"].shape), off)})
            torch.cuda.synchronize()
            for k in KEYS:
                assert torch.equal(out[k], ref[k]), (tune, k)


@pytest.mark.parametrize("dtype", ["u16", "f32"])
@pytest.mark.parametrize("shape,off", [((8, 1029, 2047), 0), ((8, 1029, 2047), 1),
                                       ((3, 2075, 1000), 1)])
def test_general_row_bands(shape, off, dtype):
    """A paced frame with more tiles than resident workgroups goes out as bands
    of rows; here their first rows start at odd elements of stack and volume."""
    st = _stack(shape, dtype, off)
    geo = (35.0, 0.4, 0.115)
    ref = dsk.deskew(st, *geo, tune=SCALAR)
    assert shape[1] * (-(-ref["width"] // 256)) > 32 * 256
    for tune in (dict(block=64, per_thread=4, unroll=2, pace_gbs=5000),
                 dict(block=64, per_thread=4, unroll=4, pace_gbs=5700)):
        out = dsk.deskew(st, *geo, tune=tune, out={"vol": _volume(tuple(ref["vol"].shape), off)})
        torch.cuda.synchronize()
        for k in KEYS:
            assert torch.equal(out[k], ref[k]), (tune, k)
