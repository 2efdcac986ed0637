"""The column stretch over few rows and columns."""
import pytest
import torch

import paper_2211_00645_amd as dsk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("rows,w_in", [(1, 1), (5, 7), (9, 33), (3, 300), (4, 1000), (1000, 20)])
@pytest.mark.parametrize("factor", [0.37, 1.0, 2.6])
def test_stretch_small_and_ragged(rows, w_in, factor):
    """Row groups and column blocks with remainders against the definition."""
    g = torch.Generator().manual_seed(rows)
    p = torch.rand((rows, w_in), generator=g).to(DEV)
    out = dsk.stretch(p, factor)
    torch.cuda.synchronize()
    u = torch.arange(out.shape[1], dtype=torch.float64, device=DEV) / factor
    i = torch.floor(u)
    f, i = u - i, i.long().clamp(max=w_in)
    pad = torch.cat([p.double(), torch.zeros((rows, 2), dtype=torch.float64, device=DEV)], 1)
    ref = (1 - f) * pad[:, i] + f * pad[:, i + 1]
    # two weights and two operations rounded to float32
    assert bool(((out.double() - ref).abs() <= 4 * 2.0 ** -24 * ref).all())
