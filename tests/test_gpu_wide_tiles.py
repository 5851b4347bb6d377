"""Ragged slots on the 256 x 256 tiles of the bf16 GEMMs.  Small launches take 64 x 64 tiles, so these have three
column tiles and 64 slots in every GEMM, 171 wide tiles by the dispatch's estimate against its 96
(test_host_routes.py holds them to that)."""
import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz
from oracle import moe_backward as ob
from oracle import moe_layer as om
from workloads import f32_to_bf16_bits

from gpu_util import to_dev, to_host
from test_gpu_narrow_tiles import _run

pytestmark = pytest.mark.gpu

# K of 520 and 584: partial last steps in every GEMM; 768 and 576: whole steps, an odd and an even number of them
SIZES = [(520, 584), (768, 576)]
# the four 64-row classes of a last tile at their edges, whole tiles, one-row and empty slots
COUNTS = [0, 1, 63, 64, 65, 127, 128, 129, 190, 192, 193, 255, 256, 257, 300, 10] * 4


def _row_by_row(got, ref, what):
    """The bf16 bar (2e-2 of the largest value), of each row by itself: a tail row must not hide behind the others."""
    err = np.max(np.abs(om.widen(got) - ref), axis=1)
    assert np.all(err <= 2e-2 * np.max(np.abs(ref), axis=1) + 1e-6), (what, np.argmax(err))


@pytest.mark.parametrize("act", ["gelu", "swiglu"])
@pytest.mark.parametrize("d,ffn", SIZES)
def test_ragged_slots_on_wide_tiles(act, d, ffn):
    S, P = len(COUNTS), sum(COUNTS)
    code = lz.LZ_GELU if act == "gelu" else lz.LZ_SWIGLU
    rng = np.random.default_rng(d)
    n1 = ffn * (2 if act == "swiglu" else 1)
    w1 = to_dev(f32_to_bf16_bits((0.05 * rng.standard_normal((S, d, n1))).astype(np.float32)), True)
    w2 = to_dev(f32_to_bf16_bits((0.05 * rng.standard_normal((S, ffn, d))).astype(np.float32)), True)
    xh = f32_to_bf16_bits(rng.standard_normal((P, d)).astype(np.float32))
    x, off, slots = to_dev(xh, True), np.concatenate([[0], np.cumsum(COUNTS)]), np.arange(S)
    w1h, w2h = to_host(w1).transpose(0, 2, 1), to_host(w2).transpose(0, 2, 1)
    yp_ref = om.expert_ffn_rows(xh, off, slots, w1h, w2h, act)

    yp, fused = _run(code, d, ffn, COUNTS, x, w1, w2, False)
    assert np.array_equal(yp, fused)
    _row_by_row(yp, yp_ref, "yp")

    first = _run(code, d, ffn, COUNTS, x, w1, w2, True)
    for _ in range(3):   # the trailing loads of one wave and the patches of another share LDS: every run the same bits
        for a, b in zip(first, _run(code, d, ffn, COUNTS, x, w1, w2, True)):
            assert np.array_equal(a, b)
    z, h, yp, dxp = first
    z_ref = np.concatenate([om.widen(xh[a:b]) @ om.widen(w1h[s]).T for s, a, b in zip(slots, off, off[1:])])
    _row_by_row(z, z_ref, "z")
    _row_by_row(h, ob.act_forward(z_ref, act), "h")
    _row_by_row(yp, yp_ref, "yp of the training forward")
    _row_by_row(dxp, ob.ffn_backward_rows(yp, xh, off, slots, w1h, w2h, act)[0], "dxp")   # dyp = yp
