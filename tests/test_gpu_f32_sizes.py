"""The fp32 matrix-core GEMM at the edges of its tiles: 32-row parts, partial stages and columns, 16-byte pieces and
single elements, both wave layouts.  The fp32 bar of the layer (1e-5 of the largest value) throughout."""
import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz
from oracle import moe_layer as om
from workloads import CONFIGS
from workloads.configs import scaled

from gpu_util import DEV, to_dev, to_host
from test_gpu_backward import _layer_backward_generic
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
