"""Small batches on 64 x 64 tiles: the same bits as the same rows inside a batch that takes the wide tiles."""
import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz
from oracle import moe_layer as om
from workloads import f32_to_bf16_bits

from gpu_util import DEV, to_dev, to_host

pytestmark = pytest.mark.gpu


def _run(act, d, ffn, counts, xrows, w1, w2, train):
    """Forward (and with `train` also data gradients) of `counts` rows per slot; all results as bf16 bits."""
    P = int(sum(counts))
    shape = lz.Shape(P, d, ffn, len(counts), 1, 1, len(counts), lz.LZ_BF16, act)
    off = to_dev(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32))
    bf = dict(dtype=torch.bfloat16, device=DEV)
    yp, dxp = torch.zeros((P, d), **bf), torch.zeros((P, d), **bf)
    n1 = ffn * (2 if act == lz.LZ_SWIGLU else 1)
    if not train:
        n = lz.lz_ffn_workspace_bytes(shape)
        ws = torch.empty(n, dtype=torch.uint8, device=DEV)
        for _ in range(2):  # the table is built anew each time
            lz.lz_expert_ffn(xrows, off, w1, w2, shape, yp, ws, n)
        fused = torch.zeros_like(yp)
        ident = torch.arange(P, dtype=torch.int32, device=DEV)
        lz.lz_expert_ffn_gather(xrows, ident, off, w1, w2, shape, fused, ws, n)
        return [to_host(yp), to_host(fused)]
    n = lz.lz_train_workspace_bytes(shape)
    ws = torch.empty(n, dtype=torch.uint8, device=DEV)
    z, h = torch.zeros((P, n1), **bf), torch.zeros((P, ffn), **bf)
    dw1, dw2 = torch.zeros_like(w1), torch.zeros_like(w2)
    lz.lz_ffn_forward_train(xrows, off, w1, w2, shape, z, h, yp, ws, n)
    lz.lz_ffn_backward(yp, xrows, z, h, off, w1, w2, shape, dxp, dw1, dw2, ws, n)
    return [to_host(t) for t in (z, h, yp, dxp)]


@pytest.mark.parametrize("train", [False, True])
@pytest.mark.parametrize("act", [lz.LZ_GELU, lz.LZ_SWIGLU])
@pytest.mark.parametrize("d,ffn", [(64, 64), (264, 200), (512, 328), (1024, 520)])
def test_small_batch_has_the_bits_of_a_large_one(act, d, ffn, train):
    counts = [63, 0, 65, 1, 64, 130]                # below, at and above a tile, empty and one-row slots
    rng = np.random.default_rng(d + ffn)
    n1 = ffn * (2 if act == lz.LZ_SWIGLU else 1)
    w1 = to_dev(f32_to_bf16_bits((0.05 * rng.standard_normal((6, d, n1))).astype(np.float32)), True)
    w2 = to_dev(f32_to_bf16_bits((0.05 * rng.standard_normal((6, ffn, d))).astype(np.float32)), True)
    P = sum(counts)
    x = rng.standard_normal((P, d)).astype(np.float32)
    small = _run(act, d, ffn, counts, to_dev(f32_to_bf16_bits(x), True), w1, w2, train)
    # each slot's rows at the head of a slot of some 5000: enough wide tiles in every GEMM
    big, at, heads = [], 0, []
    for c in counts:
        heads.append(sum(len(b) for b in big))
        big.append(np.concatenate([x[at:at + c], rng.standard_normal((5000, d)).astype(np.float32)]))
        at += c
    large = _run(act, d, ffn, [len(b) for b in big], to_dev(f32_to_bf16_bits(np.concatenate(big)), True), w1, w2, train)
    rows = np.concatenate([np.arange(a, a + c) for a, c in zip(heads, counts)])
    for s, l in zip(small, large):
        assert np.any(s)
        assert np.array_equal(s, l[rows])
    if not train:
        ref = om.expert_ffn_rows(f32_to_bf16_bits(x), np.concatenate([[0], np.cumsum(counts)]), np.arange(6),
                                 to_host(w1).transpose(0, 2, 1), to_host(w2).transpose(0, 2, 1),
                                 "gelu" if act == lz.LZ_GELU else "swiglu")
        assert np.max(np.abs(om.widen(small[0]) - ref)) <= 2e-2 * np.max(np.abs(ref))
