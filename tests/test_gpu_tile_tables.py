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


def _round_up(n, to):
    return -(-n // to) * to


def _tile_rows(counts, d, ffn, act):
    """Rows of a tile in the two GEMMs' unit tables, from the forward's workspace: hidden, then a table of the first GEMM and
    one of the second; 0: none (narrow tiles)."""
    S, P = len(counts), sum(counts)
    c = next(c for c in range(64, 0, -1) if S % c == 0)
    shape = lz.Shape(P, d, ffn, 1, 1, S // c, c, lz.LZ_BF16, act)
    n = lz.lz_ffn_workspace_bytes(shape)
    ws = torch.zeros(n, dtype=torch.uint8, device=DEV)
    lz.lz_ffn_tiles(to_dev(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)), shape, ws, n)
    ints = ws.cpu().numpy().view(np.int32)
    up = _round_up(P * ffn * 2, 256) // 4
    units = -(-(P // 256 + S) * -(-_columns(d, ffn, act)[0] // 8) // 8)            # of an XCD's list; 8 ints each, after a
    down = up + _round_up((64 + 17 * 32 + 8 * 8 * units) * 4, 256) // 4             # header of 64 ints and 17 lines of counters
    return [int(ints[up + 16]), int(ints[down + 16])]


def _columns(d, ffn, act):
    return -(-ffn // (128 if act == lz.LZ_SWIGLU else 256)), -(-d // 256)


def _first_to_end(counts, n_tiles):
    """The height with which N tiles on the CUs end first: ceil(N / CUs) rounds of a tile's mean cost, a lower one only
    if it gains 5 %."""
    cost, cus = {0: 0, 1: 50, 2: 65, 3: 82, 4: 100}, torch.cuda.get_device_properties(0).multi_processor_count // 8 * 8
    if sum(counts) / 256 * n_tiles > 16 * cus:
        return 256
    best = None
    for h in (4, 3, 2, 1):
        tiles = sum(-(-n // (64 * h)) for n in counts)
        total = sum(n // (64 * h) * cost[h] + cost[-(-(n % (64 * h)) // 64)] for n in counts)
        time = -(-tiles * n_tiles // cus) * total / tiles
        if best is None or time < 0.95 * best[0]:
            best = time, 64 * h
    return best[1]


@pytest.mark.parametrize("counts,d,ffn,act,want", [
    ([683] * 60, 264, 2600, lz.LZ_SWIGLU, [256, 192]),        # the three of test_units_of_the_persistent_kernel
    ([300, 301] * 15, 264, 2600, lz.LZ_SWIGLU, [256, 128]),
    ([130] * 3, 264, 2600, lz.LZ_SWIGLU, [64, 0]),
    ([130] * 40, 768, 768, lz.LZ_GELU, [128, 128]),
    ([400] * 12, 2600, 2600, lz.LZ_GELU, [192, 192]),
    ([16384], 4096, 4096, lz.LZ_GELU, [256, 256]),
    ([0, 1, 63, 65, 129, 191, 193, 255, 257, 700] * 6, 768, 1304, lz.LZ_GELU, None),
    ([(37 * i) % 500 for i in range(1024)], 512, 512, lz.LZ_GELU, None),
])
def test_tile_heights(counts, d, ffn, act, want):
    got = _tile_rows(counts, d, ffn, act)
    model = [_first_to_end(counts, n) if g else 0 for n, g in zip(_columns(d, ffn, act), got)]
    assert got == model and any(got)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert want is None or got == want
