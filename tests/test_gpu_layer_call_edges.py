"""A layer's passes in one call on buffers past their alignment, without rows and with flagged plans: the bits of the single calls."""
import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz

from gpu_util import DEV
from test_gpu_layer_calls import BACKWARD, FORWARD, _pair

pytestmark = pytest.mark.gpu


def _same(a, b, names):
    for name in names:
        x, y = getattr(a, name), getattr(b, name)
        width = torch.int32 if x.element_size() == 4 else torch.int16       # (an unaligned view has no bytes of its own)
        assert torch.equal(x.view(width), y.view(width)), name


def _check_passes(one, single, logits, x, dy):
    for layer in (one, single):
        layer.forward(logits, x)
    _same(one, single, FORWARD)
    for layer in (one, single):
        layer.y.zero_()
        layer.forward_fused(logits, x)
    _same(one, single, FORWARD)
    for layer in (one, single):
        layer.forward_train(logits, x)
        layer.backward(dy)
    _same(one, single, FORWARD + BACKWARD + ("dw1_slot", "dw2_slot", "dw1", "dw2"))
    for layer in (one, single):
        layer.forward_train(logits, x)
        layer.backward_accumulate(dy)
    _same(one, single, BACKWARD + ("dw1_acc", "dw2_acc"))


@pytest.mark.parametrize("dtype", [lz.LZ_F32, lz.LZ_BF16])
@pytest.mark.parametrize("names", [("w1",), ("xp",), ("z",), ("h",), ("yp",), ("dyp",), ("dxp",), ("w2", "dw1_slot"), ("dw2_slot", "dx"),
                                   ("dw1_acc", "y"), ("dw1", "dw2_acc")], ids="+".join)
def test_unaligned_buffers(dtype, names):
    """An element past their 16-byte boundary, where the kernels and their tables are others: those the tables were built for."""
    (one, single), logits, x, dy = _pair(300, 96, 200, 6, 2, 3, 4, dtype, lz.LZ_SWIGLU)
    for layer in (one, single):
        for name in names:
            t = getattr(layer, name)
            moved = torch.empty(t.numel() + 1, dtype=t.dtype, device=DEV)[1:].view(t.shape)
            setattr(layer, name, moved.copy_(t))
            assert moved.data_ptr() % 16 != 0 and moved.is_contiguous()
    _check_passes(one, single, logits, x, dy)


@pytest.mark.parametrize("T", [0, 90, 5000])     # without rows; one workgroup; tables beside the placing workgroups
@pytest.mark.parametrize("fault", ["uncovered", "split", "no expert"])
def test_flagged_plans_and_empty_batches(T, fault):
    """Tables from the slots' sizes are those from the offsets that a flagged plan leaves."""
    E, N, c = 6, 3, 4
    plan = np.array([0, 1, 2, 3, 4, 5, 0, 1, 2, 3, 4, 4], dtype=np.int32)
    off = np.array([0, T // 4, T // 2, T], dtype=np.int32)
    if fault == "uncovered":
        plan[plan == 5] = 0
    if fault == "split":
        off = np.array([0, T + 9, T // 2, T + 3], dtype=np.int32)
    if fault == "no expert":
        plan[7] = E
        plan[11] = -1
    for dtype, act in ((lz.LZ_F32, lz.LZ_GELU), (lz.LZ_BF16, lz.LZ_SWIGLU)):
        (one, single), logits, x, dy = _pair(T, 256, 320, E, 2, N, c, dtype, act)
        for layer in (one, single):
            layer.set_plan(plan, off)
        _check_passes(one, single, logits, x, dy)
        if T > 0:
            assert int(one.status.item()) != 0
