"""The backward's groups of 4 columns over a block's rows: rows narrower than
a group, remainders mod 4, rows wider and narrower than the workgroup, windows
that leave the gradient volume, and unaligned buffers; against the definition
in 64 bits."""
import numpy as np
import pytest
import torch

import paper_2211_00645_amd as dsk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("off", [0, 1, 3])
@pytest.mark.parametrize("shape", [(3, 4, 1), (5, 7, 3), (4, 9, 4), (6, 300, 5), (3, 33, 62),
                                   (2, 3, 1023), (2, 5, 1030), (3, 2, 8193), (70, 40, 250)])
def test_against_definition(shape, off):
    n, r, c = shape
    g = torch.Generator().manual_seed(2)
    st = torch.rand(n * r * c + off, generator=g).to(DEV)[off:].view(shape)
    for shift, clip in ((1.3, 0), (-0.8, 3), (0.0, 1)):
        offs = np.arange(n) * shift + 0.25
        w, b = dsk.plan(shape, offsets=offs)
        w, b = max(1, w - clip), b + clip          # clipped at both ends
        gd = torch.randn(n * r * w + off, generator=g).to(DEV)[off:].view(n, r, w)
        od = torch.from_numpy(offs).to(DEV)
        t = od - b
        k = torch.floor(t)
        phi = (t - k)[:, None, None]
        at = k.long()[:, None, None] + torch.arange(c, device=DEV)
        def grad(i):
            ok = (i >= 0) & (i < w)
            v = gd.double().gather(2, i.clamp(0, w - 1).expand(n, r, c))
            return torch.where(ok.expand(n, r, c), v, 0.0)
        g0, g1 = grad(at), grad(at + 1)
        ref_in = (1 - phi) * g0 + phi * g1
        ref_off = (st.double() * (g1 - g0)).sum((1, 2))
        for kw in ({}, {"grad_offsets": False}, {"grad_in": False}):
            gi, go = dsk.backward(st, gd, od, b, **kw)
            torch.cuda.synchronize()
            if gi is not None:
                # two weights and two operations rounded to float32
                bound = ((1 - phi) * g0.abs() + phi * g1.abs()) * 4 * 2.0 ** -24
                assert bool(((gi.double() - ref_in).abs() <= bound).all()), (shape, shift, kw)
            if go is not None:
                bound = 1e-9 * 2 * float(st.max()) * gd.double().abs().sum((1, 2))
                assert bool(((go - ref_off).abs() <= bound).all()), (shape, shift, kw)
