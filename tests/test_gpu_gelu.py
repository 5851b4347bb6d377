"""GELU of the bf16 kernels at every finite bf16 number, and at infinities and NaN."""
import math

import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz
from oracle import moe_layer as om

from gpu_util import DEV, to_dev, to_host

pytestmark = pytest.mark.gpu

D = 256


def _train_forward(bits):
    """z and h of rows of bf16 bits through one slot whose weights are the identity: z is x, h gelu(x)."""
    P = len(bits)
    shape = lz.Shape(P, D, D, 1, 1, 1, 1, lz.LZ_BF16, lz.LZ_GELU)
    eye = torch.eye(D, dtype=torch.bfloat16, device=DEV).unsqueeze(0).contiguous()
    z, h, yp = (torch.zeros((P, D), dtype=torch.bfloat16, device=DEV) for _ in range(3))
    n = lz.lz_train_workspace_bytes(shape)
    ws = torch.empty(n, dtype=torch.uint8, device=DEV)
    lz.lz_ffn_forward_train(to_dev(bits, True), to_dev(np.array([0, P], dtype=np.int32)), eye, eye, shape, z, h, yp, ws, n)
    n = lz.lz_ffn_workspace_bytes(shape)
    ws = torch.empty(n, dtype=torch.uint8, device=DEV)
    lz.lz_expert_ffn(to_dev(bits, True), to_dev(np.array([0, P], dtype=np.int32)), eye, eye, shape, yp, ws, n)
    return to_host(z), to_host(h), to_host(yp)


@pytest.mark.parametrize("copies", [1, 100])     # narrow tiles, wide tiles
def test_every_finite_number(copies):
    bits = np.arange(1 << 16, dtype=np.uint32).astype(np.uint16).reshape(256, D)
    bits = np.where((bits & 0x7F80) == 0x7F80, np.uint16(0), bits)
    v = om.widen(bits).astype(np.float64)
    exact = v * 0.5 * np.vectorize(math.erfc)(-v / math.sqrt(2.0))
    z, h, yp = _train_forward(np.tile(bits, (copies, 1)))
    # half a bf16 step, and 4e-7 of the formula in fp32 (3.1e-7 of its fit and roundings on [-8, 8]; past that relative to v)
    _, e = np.frexp(exact)
    bar = np.ldexp(1.0, e - 9) + 4e-7 + 1.2e-7 * np.abs(v)
    for c in range(copies):
        rows = slice(256 * c, 256 * c + 256)
        assert np.array_equal(om.widen(z[rows]), om.widen(bits))
        for got in (h[rows], yp[rows]):
            assert np.all(np.abs(om.widen(got) - exact) <= bar)


@pytest.mark.parametrize("copies", [1, 100])
def test_infinities_and_nan(copies):
    """One of them a row: +inf stays, -inf gives the NaN of inf - inf, as the definition in floats does."""
    bits = np.zeros((256, D), dtype=np.uint16)
    special = [0x7F80, 0xFF80, 0x7FC0]
    for i, b in enumerate(special):
        bits[i, 3 + i] = b
    _, h, _ = _train_forward(np.tile(bits, (copies, 1)))
    h = om.widen(h).reshape(copies, 256, D)
    assert np.all(h[:, 0, 3] == np.inf)
    assert np.all(np.isnan(h[:, 1, 4])) and np.all(np.isnan(h[:, 2, 5]))
    assert np.all(h[:, 3:] == 0)
