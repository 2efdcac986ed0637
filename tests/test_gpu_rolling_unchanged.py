"""Rolling update where only part of a frame changes: planes of every length
mod 4, images replaced by themselves, by others and back, and projections
handed in as new buffers; bitwise the deskew of the stack the view holds."""
import pytest
import torch

import paper_2211_00645_amd as dsk
from paper_2211_00645_amd.rolling import RollingView

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("shape", [(5, 3, 7), (9, 1, 2), (17, 5, 40), (1, 3, 11), (6, 7, 64)])
def test_partly_changed_frames(shape):
    n, r, c = shape
    g = torch.Generator().manual_seed(3)
    a, b = (torch.randint(0, 65536, shape, generator=g, dtype=torch.int32).to(torch.uint16).to(DEV)
            for _ in range(2))
    b[:, r // 2:] = a[:, r // 2:]            # half of every image stays
    rv = RollingView(*shape, 35.0, 0.4, 0.115)
    cur = a.clone()
    for i in range(n):
        rv.update(i, a[i])
    for i, src in [(0, b), (n - 1, b), (n // 2, a), (n // 2, b), (0, a), (n - 1, b)]:
        rv.psum = torch.full_like(rv.psum, float("nan"))
        rv.pmax = torch.full_like(rv.pmax, float("nan"))
        rv.update(i, src[i])
        cur[i] = src[i]
        ref = dsk.deskew(cur, 35.0, 0.4, 0.115)
        torch.cuda.synchronize()
        assert torch.equal(rv.vol, ref["vol"]) and torch.equal(rv.pmax, ref["pmax"])
        # sums of a few 16-bit values times 24-bit weights: exact in 64 bits
        # but for their last bits, rounded once
        torch.testing.assert_close(rv.psum, ref["psum"], rtol=2.0 ** -23, atol=0)
