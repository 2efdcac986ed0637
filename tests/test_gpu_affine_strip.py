"""The affine strip kernel where it can go wrong: rows narrower than a strip,
a strip or a group past the last column, rows past the last, reversed sweeps,
bands near the ring's size, and outputs large enough that strips start at
line boundaries (rows of one phase taken apart); against the definition in
64 bits."""
import math

import pytest
import torch

import paper_2211_00645_amd as dsk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(shape, ang, step, dy, rows=None, off=0):
    n, r, c = shape
    g = torch.Generator().manual_seed(7)
    flat = torch.randint(0, 65536, (n * r * c + off,), generator=g, dtype=torch.int32)
    st = flat.to(torch.uint16).to(DEV)[off:].view(shape)
    y0, ny = dsk.affine_plan(shape, ang, step, 0.115, dy)
    vol = torch.full((ny, r, c), float("nan"), device=DEV)
    dsk.affine(st, ang, step, 0.115, dy, out=vol)
    pc = 0.115 * math.cos(ang * math.pi / 180.0)
    z = torch.arange(c, device=DEV)
    f32 = st.to(torch.int32).float()
    zero = torch.zeros((1, r, c), device=DEV)
    img = torch.cat([zero, zero, f32, zero, zero])          # image n at n + 2
    for y in rows if rows is not None else range(ny):
        u = (y0 + y * dy - z.double() * pc) / step
        i = torch.floor(u)
        f = (u - i)[:, None]
        i = i.clamp(-2, n).long() + 2
        ref = ((1.0 - f) * img[i, :, z].double() + f * img[i + 1, :, z].double()).T
        # two weights and two operations rounded to float32 (4 of 2^-24), and
        # the coordinate's own rounding: u up to 2^11 in 64 bits, times the
        # largest pixel difference
        err = (vol[y % ny].double() - ref).abs()
        assert bool((err <= 1e-6 * ref + 65536 * 2.0 ** -40).all()), (y, float(err.max()))


@pytest.mark.parametrize("shape,ang,step,dy", [
    ((9, 3, 1), 35.0, 0.4, 0.115), ((9, 5, 2), 35.0, 0.4, 0.115), ((30, 1, 3), 30.0, 0.2, 0.115),
    ((40, 4, 63), 45.0, 0.2, 0.115), ((40, 5, 64), 30.0, 0.25, 0.115),
    ((40, 6, 65), 35.0, -0.31, 0.115), ((70, 2, 127), 30.0, -0.2, 0.115),
    ((25, 7, 129), 60.0, 0.4, 0.37), ((25, 7, 130), 120.0, 0.3, 0.115),
    ((60, 3, 96), 35.0, 0.125, 0.115),        # the ring's widest bands
    ((60, 3, 96), 35.0, 0.11, 0.115),         # and past them
])
@pytest.mark.parametrize("off", [0, 1])
def test_small(shape, ang, step, dy, off):
    _check(shape, ang, step, dy, off=off)


@pytest.mark.parametrize("shape,ang,step,dy", [
    ((60, 131, 333), 45.0, 0.23, 0.0085),     # rows 32 apart, the last class short
    ((40, 70, 1002), 30.0, -0.3, 0.012),      # rows 16 apart, reversed
    ((60, 37, 1100), 35.0, 0.4, 0.015),       # rows 8 apart
    ((60, 66, 992), 35.0, 0.4, 0.025),        # whole lines
])
def test_large_outputs(shape, ang, step, dy):
    _, ny = dsk.affine_plan(shape, ang, step, 0.115, dy)
    assert 4 * ny * shape[1] * shape[2] > 256000000
    _check(shape, ang, step, dy, rows=[*range(0, 40), *range(250, 290), ny // 2,
                                       *range(ny - 40, ny)])


@pytest.mark.parametrize("shape,ang,step,dy", [
    ((70, 5, 129), 35.0, 0.4, 0.38),          # 15.2 images a chunk
    ((70, 3, 200), 30.0, 0.4, 0.3996),        # 15.98
    ((70, 3, 66), 60.0, -0.4, 0.399),         # reversed
    ((600, 330, 301), 45.0, 0.38, 0.38 * 0.999),   # rows of one phase apart
])
@pytest.mark.parametrize("off", [0, 1])
def test_steps_nearly_as_coarse_as_the_scan(shape, ang, step, dy, off):
    """Up to 16 new images a chunk of 16 y values."""
    _, ny = dsk.affine_plan(shape, ang, step, 0.115, dy)
    rows = None if ny < 200 else [*range(0, 40), ny // 2, *range(ny - 40, ny)]
    _check(shape, ang, step, dy, rows=rows, off=off)
