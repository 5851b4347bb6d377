"""Replica sums of the weight gradients: the 16-byte kernel's edges and the element-wise kernel beside it."""
import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz
from oracle import moe_backward as ob
from oracle import moe_layer as om
from workloads import f32_to_bf16_bits

from gpu_util import DEV, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("S,E,n", [(1, 1, 8), (64, 5, 4088), (65, 3, 4096), (130, 67, 8200), (7, 4, 4099),
                                   (5, 2, 1020), (5, 2, 1028), (5, 2, 2040), (5, 2, 2056), (200, 3, 1032)])
def test_replica_sums(dtype, S, E, n):
    """Slots in more than one group of 64, an expert without a slot, vector counts around a block's 256, more and
    fewer of an expert's slots than are loaded ahead, and sizes that are no whole number of 16-byte vectors.  An fp32 sum of r terms is off by at most (r - 1) 2^-24
    of the sum of their absolute values; a bf16 result by half a bf16 step (2^-9) more."""
    rng = np.random.default_rng(S + n)
    plan = rng.integers(0, max(1, E - 1), size=S).astype(np.int32)   # the last expert has no slot (E > 1)
    dws = rng.standard_normal((S, n)).astype(np.float32)
    src = dws if dtype == "f32" else f32_to_bf16_bits(dws)
    dw = torch.full((E, n), 5.0, dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device=DEV)
    lz.lz_reduce_replica_grads_dtype(to_dev(src, dtype == "bf16"), to_dev(plan), S, E, n,
                                     lz.LZ_F32 if dtype == "f32" else lz.LZ_BF16, dw)
    wide = om.widen(src)
    ref, mag = ob.reduce_replica_grads(wide, plan, E), ob.reduce_replica_grads(np.abs(wide), plan, E)
    bound = S * 2.0 ** -24 * mag + (0 if dtype == "f32" else 2.0 ** -8 * np.abs(ref))
    assert np.all(np.abs(om.widen(to_host(dw)) - ref) <= bound)
