"""The fp32 matrix-core GEMM at the edges of its tiles: 32-row parts, partial stages and columns, 16-byte pieces and
single elements, both wave layouts.  The fp32 bar of the layer (1e-5 of the largest value) throughout."""
import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz
from oracle import moe_backward as ob
from oracle import moe_layer as om
from workloads import CONFIGS, f32_to_bf16_bits
from workloads.configs import scaled

from gpu_util import DEV, to_dev, to_host
from test_gpu_backward import _layer_backward_generic, test_weight_gradients_accumulate_in_fp32_over_micro_batches as accumulate_case
from test_gpu_fused_gather import _case as fused_case
from test_gpu_parity import _ffn_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act", ["gelu", "swiglu"])
@pytest.mark.parametrize("d,ffn", [(1, 1), (3, 5), (4, 4), (63, 65), (64, 60), (132, 36), (127, 260)])
def test_ffn_f32_sizes(act, d, ffn):
    cfg = scaled(CONFIGS["c1_tiny"], act=act, T=150, k=2, d=d, ffn=ffn, N=3, c=2)
    assert _ffn_case(cfg, [31, 0, 1, 170, 33, 65], 1) <= 1e-5
    assert fused_case(cfg, [64, 32, 96, 0, 95, 13], 2) <= 1e-5


@pytest.mark.parametrize("act,d,ffn", [("gelu", 40, 1040), ("swiglu", 36, 530), ("gelu", 1030, 31), ("swiglu", 33, 1029)])
def test_layer_f32_wide(act, d, ffn):
    """More than 3072 tiles of 32 x 32 in one GEMM or another: the layout of four waves side by side."""
    cfg = scaled(CONFIGS["c1_tiny"], act=act, T=1500, d=d, ffn=ffn, E=8, k=2, N=3, c=4,
                 replica_counts=(2, 2, 2, 2, 1, 1, 1, 1))
    _layer_backward_generic(cfg, 1e-5)


# d, ffn, slots: 3072 tiles of 32 x 32 and more in both weight gradients, in 16-byte pieces and in elements
WIDE_GRADIENTS = [(512, 512, 12), (511, 509, 12), (448, 448, 16), (447, 445, 16)]


@pytest.mark.parametrize("d,ffn", [w[:2] for w in WIDE_GRADIENTS[:2]])
def test_layer_f32_wide_weight_gradients(d, ffn):
    """Weight gradients on four waves side by side (test_host_routes.py holds these sizes to that)."""
    cfg = scaled(CONFIGS["c1_tiny"], T=300, d=d, ffn=ffn, E=8, k=2, N=3, c=4, replica_counts=(2, 2, 2, 2, 1, 1, 1, 1))
    _layer_backward_generic(cfg, 1e-5)


@pytest.mark.parametrize("d,ffn", [w[:2] for w in WIDE_GRADIENTS[2:]])
def test_accumulated_f32_wide_weight_gradients(d, ffn):
    accumulate_case("f32", d, ffn, "gelu")


@pytest.mark.parametrize("act", ["gelu", "swiglu"])
def test_bf16_rows_of_no_whole_pieces(act):
    """bf16 widths that are no multiple of 8 run on the fp32 kernel too: both forwards, training, accumulation."""
    cfg = scaled(CONFIGS["c1_tiny"], act=act, dtype="bf16", T=150, k=2, d=71, ffn=205, N=3, c=2)
    assert _ffn_case(cfg, [31, 0, 1, 170, 33, 65], 1) <= 2e-2
    assert fused_case(cfg, [64, 32, 96, 0, 95, 13], 2) <= 2e-2
    cfg = scaled(CONFIGS["c1_tiny"], act=act, dtype="bf16", T=333, d=71, ffn=205, E=8, k=3, N=3, c=4,
                 replica_counts=(2, 2, 2, 2, 1, 1, 1, 1))
    _layer_backward_generic(cfg, 2e-2)
    accumulate_case("bf16", 71, 205, act)


@pytest.mark.parametrize("act", ["gelu", "swiglu"])
@pytest.mark.parametrize("accumulate", [False, True])
def test_unaligned_bf16_backward(act, accumulate):
    """Widths that are multiples of 8 but no tile's: aligned tensors on the bf16 kernels, unaligned ones on the fp32
    kernel, each tensor in turn and all of them.  Both round dZ and the stored gradients once to bf16 (2^-9
    each, dH once more on the bf16 kernels), far inside the bf16 bar."""
    T, d, ffn = 333, 264, 200
    code = lz.LZ_GELU if act == "gelu" else lz.LZ_SWIGLU
    n1 = ffn * (2 if act == "swiglu" else 1)
    shape = lz.Shape(T, d, ffn, 3, 1, 1, 3, lz.LZ_BF16, code)
    rng = np.random.default_rng(9)
    slots = np.array([0, 300, 300, T], dtype=np.int32)
    bits = lambda a: f32_to_bf16_bits(a.astype(np.float32))  # noqa: E731
    w1, w2 = bits(0.05 * rng.standard_normal((3, d, n1))), bits(0.05 * rng.standard_normal((3, ffn, d)))
    xp, dyp = bits(rng.standard_normal((T, d))), bits(rng.standard_normal((T, d)))
    zr = np.concatenate([om.widen(xp[a:b]) @ om.widen(w1[s]) for s, (a, b) in enumerate(zip(slots, slots[1:]))])
    z = bits(zr)
    h = bits(ob.act_forward(om.widen(z), act))
    ref = ob.ffn_backward_rows(dyp, xp, slots, np.arange(3), w1.transpose(0, 2, 1), w2.transpose(0, 2, 1), act)
    refs = [ref[0], ref[1].transpose(0, 2, 1), ref[2].transpose(0, 2, 1)]
    ws = torch.empty(lz.lz_train_workspace_bytes(shape), dtype=torch.uint8, device=DEV)
    off = to_dev(slots)

    def placed(a, shift):
        buf = torch.zeros(a.size + 1, dtype=torch.bfloat16 if a.dtype == np.uint16 else torch.float32, device=DEV)
        v = buf[shift:shift + a.size].view(a.shape)
        v.copy_(to_dev(a, a.dtype == np.uint16))
        return v

    host = [dyp, xp, z, h, w1, w2, np.zeros((T, d), np.uint16)]
    host += [np.zeros((3, d, n1), np.float32 if accumulate else np.uint16), np.zeros((3, ffn, d), np.float32 if accumulate else np.uint16)]
    for odd in [(), tuple(range(9)), *((i,) for i in range(9))]:
        t = [placed(a, i in odd) for i, a in enumerate(host)]
        call = lz.lz_ffn_backward_accumulate if accumulate else lz.lz_ffn_backward
        call(*t[:4], off, t[4], t[5], shape, *t[6:], ws, ws.numel())
        for got, want in zip(t[6:], refs):
            got = got.float().cpu().numpy()
            assert np.max(np.abs(got - want)) <= 2e-2 * np.max(np.abs(want)), odd
        assert not t[7][1].any() and not t[8][1].any()     # the empty slot


@pytest.mark.parametrize("off", [1, 2, 3])
def test_f32_unaligned_tensors_give_the_aligned_bits(off):
    T, d, ffn = 100, 68, 36
    shape = lz.Shape(T, d, ffn, 2, 1, 1, 2, lz.LZ_F32, lz.LZ_SWIGLU)
    rng = np.random.default_rng(8)

    def at(a, shift):
        buf = torch.zeros(a.size + 4, dtype=torch.float32, device=DEV)
        v = buf[shift:shift + a.size].view(a.shape)
        v.copy_(to_dev(a.astype(np.float32)))
        return v

    a = [rng.standard_normal((T, d)), 0.1 * rng.standard_normal((2, d, 2 * ffn)), 0.1 * rng.standard_normal((2, ffn, d))]
    slots = to_dev(np.array([0, 61, T], dtype=np.int32))
    n = lz.lz_ffn_workspace_bytes(shape)
    ws = torch.empty(n, dtype=torch.uint8, device=DEV)
    out = []
    for s in (0, off):
        yp = at(np.zeros((T, d)), s)
        lz.lz_expert_ffn(at(a[0], s), slots, at(a[1], s), at(a[2], s), shape, yp, ws, n)
        out.append(to_host(yp.contiguous()))
    assert np.array_equal(out[0], out[1]) and np.all(np.isfinite(om.widen(out[0])))
