"""The row-tile tables the grouped GEMMs draw their work from, on offsets that strain them."""
import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz

from gpu_util import DEV, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log_P", [12, 25])
def test_offsets_that_fall_again_stay_inside_the_table(log_P):
    """Offsets 0, P, 0, P, ... clip to overlapping slots: S / 2 of them with all P rows each, from 2^25 rows on more
    32-row tiles than an int counts.  The table ends at its capacity (P / 32 + S tiles: all of slot 0 and the head of
    slot 2) and nothing is written past the workspace."""
    P, S = 1 << log_P, 4096
    shape = lz.Shape(P, 1, 1, 1, 1, 64, 64, lz.LZ_F32, lz.LZ_GELU)
    off = to_dev(np.where(np.arange(S + 1) % 2 == 0, 0, P).astype(np.int32))
    n, guard = lz.lz_ffn_workspace_bytes(shape), 1 << 20
    ws = torch.full((n + guard,), 0x5A, dtype=torch.uint8, device=DEV)
    x = torch.linspace(-2, 2, P, device=DEV).view(P, 1)
    ones = torch.ones((S, 1, 1), device=DEV)       # every slot the same weights: an overlap does not show in y
    yp = torch.full((P, 1), 7.0, device=DEV)
    lz.lz_expert_ffn(x, off, ones, ones, shape, yp, ws, n)
    torch.cuda.synchronize()
    assert bool((ws[n:] == 0x5A).all())
    assert float((yp - torch.nn.functional.gelu(x)).abs().max()) <= 1e-6   # |gelu| <= 2: a few fp32 roundings
