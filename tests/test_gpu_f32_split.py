"""The fp32 GEMM on split operands: the sizes that it takes (two 64 x 128 tiles a CU and more), at the edges of tiles,
stages and fragments, against fp64.  Bound: the products are exact to 2^-30, the sum is rounded at most three times in 32 k,
a random walk of 3 K / 32 roundings of 2^-24: 2e-6 of the largest value at K <= 1500."""
import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz

from gpu_util import DEV

pytestmark = pytest.mark.gpu
BOUND = 2e-6


def _slots(rng, S, P):
    cuts = np.sort(rng.integers(0, P + 1, S - 1))
    cuts[2] = cuts[1]                      # an empty slot
    return np.concatenate([[0], np.sort(cuts), [P]]).astype(np.int32)


def _act(z, ffn, act):
    return torch.nn.functional.gelu(z) if act == "gelu" else torch.nn.functional.silu(z[:, :ffn]) * z[:, ffn:]


def _close(got, want, bound=BOUND):
    assert got.shape == want.shape
    assert float((got.double() - want).abs().max()) <= bound * float(want.abs().max())


# up and down projection and both gradients on split operands: 20 slots, 2400 rows (47 row tiles), 512 tiles and more
@pytest.mark.parametrize("act", ["gelu", "swiglu"])
@pytest.mark.parametrize("d,ffn", [(1408, 1408), (1400, 1456), (1412, 1500)])
def test_split_gemms_against_fp64(act, d, ffn):
    rng = np.random.default_rng(d + ffn)
    S, P, n1 = 20, 2400, ffn * (2 if act == "swiglu" else 1)
    shape = lz.Shape(P, d, ffn, S, 1, 1, S, lz.LZ_F32, lz.LZ_GELU if act == "gelu" else lz.LZ_SWIGLU)
    gen = torch.Generator(device=DEV).manual_seed(d)
    normal = lambda *s: torch.randn(s, generator=gen, device=DEV)  # noqa: E731
    slots = _slots(rng, S, P)
    off = torch.from_numpy(slots).to(DEV)
    x, dyp, w1, w2 = normal(P, d), normal(P, d), 0.03 * normal(S, d, n1), 0.03 * normal(S, ffn, d)
    yp, z, h, yt, dxp = (torch.empty((P, n), device=DEV) for n in (d, n1, ffn, d, d))
    dw1, dw2 = torch.full_like(w1, 7.0), torch.full_like(w2, 7.0)
    acc1, acc2 = normal(S, d, n1), normal(S, ffn, d)
    start1, start2 = acc1.double(), acc2.double()
    ws = torch.empty(max(lz.lz_ffn_workspace_bytes(shape), lz.lz_train_workspace_bytes(shape)), dtype=torch.uint8, device=DEV)
    lz.lz_expert_ffn(x, off, w1, w2, shape, yp, ws, ws.numel())
    lz.lz_ffn_forward_train(x, off, w1, w2, shape, z, h, yt, ws, ws.numel())
    lz.lz_ffn_backward(dyp, x, z, h, off, w1, w2, shape, dxp, dw1, dw2, ws, ws.numel())
    lz.lz_ffn_backward_accumulate(dyp, x, z, h, off, w1, w2, shape, dxp, acc1, acc2, ws, ws.numel())
    assert torch.equal(yp, yt)
    for s in range(S):
        a, b = slots[s], slots[s + 1]
        if a == b:
            assert not dw1[s].any() and not dw2[s].any()
            assert torch.equal(acc1[s].double(), start1[s]) and torch.equal(acc2[s].double(), start2[s])
            continue
        zs = (x[a:b].double() @ w1[s].double()).requires_grad_(True)
        hs = _act(zs, ffn, act)
        _close(z[a:b], zs.detach())
        _close(h[a:b], hs.detach())
        _close(yp[a:b], hs.detach() @ w2[s].double())
        dh = dyp[a:b].double() @ w2[s].double().T
        hs.backward(dh)
        g1, g2 = x[a:b].double().T @ zs.grad, hs.detach().T @ dyp[a:b].double()
        # dZ, an input of dw1, comes from the fp32 instruction: 8 roundings in 32 k
        _close(dw1[s], g1, 2 * BOUND)
        _close(dw2[s], g2)
        _close(acc1[s], start1[s] + g1, 2 * BOUND)
        _close(acc2[s], start2[s] + g2)


def _forward(x, w1, w2):
    P, d = x.shape
    S, _, ffn = w1.shape
    shape = lz.Shape(P, d, ffn, S, 1, 1, S, lz.LZ_F32, lz.LZ_GELU)
    off = torch.arange(0, P + 1, P // S, dtype=torch.int32, device=DEV)
    z, h, yp = (torch.empty((P, n), device=DEV) for n in (ffn, ffn, d))
    ws = torch.empty(lz.lz_train_workspace_bytes(shape), dtype=torch.uint8, device=DEV)
    lz.lz_ffn_forward_train(x, off, w1, w2, shape, z, h, yp, ws, ws.numel())
    return z


def test_split_keeps_infinities_and_nans_where_fp32_has_them():
    """Rows with infinities, NaNs and numbers near the largest: as a sum of fp32 products gives them; others untouched."""
    gen = torch.Generator(device=DEV).manual_seed(3)
    P, d, ffn, S = 2048, 128, 2048, 4
    x = torch.rand((P, d), generator=gen, device=DEV) + 0.5
    w1 = torch.rand((S, d, ffn), generator=gen, device=DEV) + 0.5
    w2 = torch.zeros((S, ffn, d), device=DEV)
    w1[0, 7, 5] = 1.0                                   # no second or third part
    clean = _forward(x, w1, w2)
    x[3, 7], x[70, 1], x[200, 9] = float("inf"), float("-inf"), float("nan")
    x[300, 1], x[300, 2] = float("inf"), float("-inf")
    x[400, 0], x[401, :] = 3.4028234e38, 3e38
    x[402, :] = 1e38 / d
    z = _forward(x, w1, w2)
    assert (z[3] == float("inf")).all() and (z[70] == float("-inf")).all()
    assert z[200].isnan().all() and z[300].isnan().all() and (z[401] == float("inf")).all()
    want = x[402].double() @ w1[0].double()
    assert z[402].isfinite().all() and float((z[402].double() - want).abs().max()) <= 1e-5 * float(want.max())
    rows = [r for r in range(P) if r not in (3, 70, 200, 300, 400, 401, 402)]
    assert float((z[rows] - clean[rows]).abs().max()) <= 1e-5 * float(clean[rows].abs().max())


@pytest.mark.parametrize("scale", [1e-30, 1e-33, 1e-36])
def test_split_of_operands_near_the_smallest_normal_number(scale):
    """Their last parts would be no normal numbers if they were split as they are."""
    gen = torch.Generator(device=DEV).manual_seed(5)
    x = torch.randn((2048, 128), generator=gen, device=DEV) * scale
    w1, w2 = torch.randn((4, 128, 2048), generator=gen, device=DEV), torch.zeros((4, 2048, 128), device=DEV)
    z = _forward(x, w1, w2)
    want = torch.cat([x[512 * s:512 * s + 512].double() @ w1[s].double() for s in range(4)])
    _close(z, want)
