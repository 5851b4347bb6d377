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


@pytest.mark.parametrize("dtype,d", [(lz.LZ_F32, 1), (lz.LZ_BF16, 8), (lz.LZ_BF16, 9)])
@pytest.mark.parametrize("counts", [
    [40000],                                            # one slot, a long list of tiles
    [0, 4 * 32, 4 * 32 + 1, 5 * 64, 1, 5 * 256 + 7, 20011, 0],
    [33] * 70 + [3000] + [0] * 60 + [161] * 69,         # long and short lists in each wave of the table's kernel
])
def test_slots_of_few_and_of_many_tiles(dtype, d, counts):
    P, S = sum(counts), len(counts)
    shape = lz.Shape(P, d, d, 1, 1, S // 50 + 1, -(-S // (S // 50 + 1)), dtype, lz.LZ_GELU)
    counts = counts + [0] * (shape.S - S)
    tdt = torch.float32 if dtype == lz.LZ_F32 else torch.bfloat16
    gen = torch.Generator(device=DEV)
    gen.manual_seed(S)
    x, w1, w2 = (torch.randn(n, generator=gen, device=DEV).to(tdt) for n in ((P, d), (shape.S, d, d), (shape.S, d, d)))
    off = to_dev(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32))
    n = lz.lz_ffn_workspace_bytes(shape)
    ws, yp = torch.empty(n, dtype=torch.uint8, device=DEV), torch.full((P, d), 7.0, dtype=tdt, device=DEV)
    lz.lz_expert_ffn(x, off, w1, w2, shape, yp, ws, n)
    slot = torch.from_numpy(np.repeat(np.arange(shape.S), counts)).to(DEV)
    h = torch.nn.functional.gelu((x.double()[:, :, None] * w1.double()[slot]).sum(1))
    ref = (h[:, :, None] * w2.double()[slot]).sum(1)
    # the layer's bars: 1e-5 in fp32, 2e-2 of the largest value in bf16
    assert float((yp.double() - ref).abs().max()) <= (1e-5 if dtype == lz.LZ_F32 else 2e-2) * float(ref.abs().max())


@pytest.mark.parametrize("counts", [
    [(7 * i) % 41 for i in range(700)],                 # 350 units a list, of few tickets each
    [0, 1029, 0, 0, 2048, 1, 255, 257, 0, 767],         # groups of 1 to 4 row tiles, some of one row
    [1] + [0] * 62 + [3],                               # fewer tiles than workgroups: most find every list empty
    [683] * 60,                                         # tiles of 192 rows in the second GEMM (on 256 CUs)
    [300, 301] * 15,                                    # of 128
    [130] * 3,                                          # of 64
])
def test_units_of_the_persistent_kernel(counts):
    """Tickets of ragged units: every tile is drawn once, and leads to its own rows and columns."""
    d, ffn, S = 264, 2600, len(counts)                  # 2 and 11 column tiles (one and two column groups)
    P, c = sum(counts), next(c for c in range(64, 0, -1) if S % c == 0)
    shape = lz.Shape(P, d, ffn, 1, 1, S // c, c, lz.LZ_BF16, lz.LZ_SWIGLU)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(S)
    x, w1, w2 = (torch.randn(n, generator=gen, device=DEV).mul_(s).bfloat16()
                 for n, s in (((P, d), 1), ((S, d, 2 * ffn), 0.1), ((S, ffn, d), 0.1)))
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    n = lz.lz_ffn_workspace_bytes(shape)
    ws = torch.empty(n, dtype=torch.uint8, device=DEV)
    out = [torch.full((P, d), 7.0, dtype=torch.bfloat16, device=DEV) for _ in range(2)]
    for yp in out:                                      # the second call draws from lists of its own
        lz.lz_expert_ffn(x, to_dev(off), w1, w2, shape, yp, ws, n)
    assert torch.equal(out[0], out[1])
    for s in np.flatnonzero(counts):
        a, b = off[s], off[s + 1]
        z = x[a:b].double() @ w1[s].double()
        ref = (torch.nn.functional.silu(z[:, :ffn]) * z[:, ffn:]) @ w2[s].double()
        assert float((out[0][a:b].double() - ref).abs().max()) <= 2e-2 * float(ref.abs().max())  # bf16 h and y
