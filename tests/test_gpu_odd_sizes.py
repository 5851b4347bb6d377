"""bf16 sizes that the MFMA tiles do not divide: partial K steps, partial column tiles, unaligned tensors."""
import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz
from oracle import moe_layer as om
from workloads import CONFIGS, f32_to_bf16_bits
from workloads.configs import scaled

from gpu_util import DEV, to_dev, to_host
from test_gpu_backward import _layer_backward_generic
from test_gpu_fused_gather import _case as fused_case
from test_gpu_parity import _ffn_case

pytestmark = pytest.mark.gpu

# K steps ending after 8, 56 and 64 of 64 columns, one short step only, one column past a tile in either GEMM
SIZES = [(8, 8), (72, 200), (264, 248), (320, 56), (520, 384), (1000, 136)]


@pytest.mark.parametrize("act", ["gelu", "swiglu"])
@pytest.mark.parametrize("d,ffn", SIZES)
def test_ffn_odd_sizes(act, d, ffn):
    cfg = scaled(CONFIGS["c1_tiny"], act=act, dtype="bf16", T=700, k=2, d=d, ffn=ffn, N=4, c=2)
    assert _ffn_case(cfg, [257, 0, 1, 512, 300, 255, 74, 1], 3) <= 2e-2       # the bf16 bar of the whole tiles
    assert fused_case(cfg, [130, 190, 65, 128, 64, 193, 400, 230], 4) <= 2e-2


@pytest.mark.parametrize("act", ["gelu", "swiglu"])
@pytest.mark.parametrize("d,ffn", [(8, 8), (264, 248), (328, 56)])
def test_layer_backward_odd_sizes(act, d, ffn):
    cfg = scaled(CONFIGS["c1_tiny"], act=act, dtype="bf16", T=333, d=d, ffn=ffn, E=8, k=3, N=3, c=4,
                 replica_counts=(2, 2, 2, 2, 1, 1, 1, 1))
    _layer_backward_generic(cfg, 2e-2)


@pytest.mark.parametrize("fused", [False, True])
def test_a_row_of_nan_stays_in_its_row(fused):
    """A partial K step ends inside a 128-byte run: what the next row holds must not get in."""
    T, d, ffn = 200, 264, 136
    shape = lz.Shape(T, d, ffn, 2, 1, 1, 2, lz.LZ_BF16, lz.LZ_SWIGLU)
    rng = np.random.default_rng(5)
    x = to_dev(f32_to_bf16_bits(rng.standard_normal((T, d)).astype(np.float32)), True)
    w1 = to_dev(f32_to_bf16_bits(0.05 * rng.standard_normal((2, d, 2 * ffn)).astype(np.float32)), True)
    w2 = to_dev(f32_to_bf16_bits(0.05 * rng.standard_normal((2, ffn, d)).astype(np.float32)), True)
    off = to_dev(np.array([0, 77, T], dtype=np.int32))
    maps = to_dev(np.arange(T, dtype=np.int32))
    n = lz.lz_ffn_workspace_bytes(shape)
    ws = torch.empty(n, dtype=torch.uint8, device=DEV)

    def ffn_of(xin):
        yp = torch.zeros((T, d), dtype=torch.bfloat16, device=DEV)
        if fused:
            lz.lz_expert_ffn_gather(xin, maps, off, w1, w2, shape, yp, ws, n)
        else:
            lz.lz_expert_ffn(xin, off, w1, w2, shape, yp, ws, n)
        return yp

    clean = ffn_of(x)
    bad = x.clone()
    bad[[1, 77, 150]] = float("nan")
    got = ffn_of(bad)
    rows = torch.ones(T, dtype=torch.bool, device=DEV)
    rows[[1, 77, 150]] = False
    assert torch.equal(got[rows].view(torch.int16), clean[rows].view(torch.int16))
    assert bool(torch.isnan(got[~rows]).all())


def test_unaligned_tensors_of_odd_sizes():
    """Odd sizes take tensors at any element offset (the fp32 kernel, with a tile table of its own)."""
    T, d, ffn = 333, 264, 200
    shape = lz.Shape(T, d, ffn, 2, 1, 1, 2, lz.LZ_BF16, lz.LZ_GELU)
    rng = np.random.default_rng(6)

    def shifted(a):
        t = to_dev(f32_to_bf16_bits(a.astype(np.float32)), True)
        buf = torch.empty(t.numel() + 1, dtype=torch.bfloat16, device=DEV)
        buf[1:] = t.reshape(-1)
        return t, buf[1:].view(t.shape)

    x, xu = shifted(rng.standard_normal((T, d)))
    w1, w1u = shifted(0.05 * rng.standard_normal((2, d, ffn)))
    w2, w2u = shifted(0.05 * rng.standard_normal((2, ffn, d)))
    off = to_dev(np.array([0, 300, T], dtype=np.int32))
    n = max(lz.lz_ffn_workspace_bytes(shape), lz.lz_train_workspace_bytes(shape))
    ws = torch.empty(n, dtype=torch.uint8, device=DEV)
    outs = []
    for a, b, c in [(x, w1, w2), (xu, w1u, w2u), (xu, w1, w2), (x, w1, w2u)]:
        yp = torch.zeros((T, d), dtype=torch.bfloat16, device=DEV)
        lz.lz_expert_ffn(a, off, b, c, shape, yp, ws, n)
        outs.append(om.widen(to_host(yp)))
    z, h = (torch.empty((T, ffn), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    yp = torch.zeros((T, d), dtype=torch.bfloat16, device=DEV)
    lz.lz_ffn_forward_train(xu, off, w1u, w2u, shape, z, h, yp, ws, n)
    outs.append(om.widen(to_host(yp)))
    for o in outs[1:]:   # both round h and yp once to bf16 (2^-9 each); a changed rounding of h moves yp by less
        assert np.max(np.abs(o - outs[0])) <= 2.0 ** -7 * np.max(np.abs(outs[0]))
