"""The fp32 GEMMs on split operands where their parts are easily lost: sums of one product, small numbers beside ordinary
ones, infinities and numbers near the largest.  20 slots, 2400 rows, two 64 x 128 tiles a CU and more: every forward GEMM and
both weight gradients run there (test_host_split_route.py holds them to that).

Bounds.  A product is rounded once, by 2^-24, and what is left out of it is below 2^-30: 2^-24 1.02.  A sum of n > 1 has n
roundings and one more, of the matrix instruction, which adds its products at the scale of the largest: (n + 1) 2^-24 1.02
of the sum of their magnitudes (found: 2.4 and 2.8 for n = 2 and 3; the fp32 instruction 1.9 and 2.5, of a larger rms).
Results below 2^-126 are multiples of 2^-149: two of those more, one for each half of the k."""
import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz

from gpu_util import DEV

pytestmark = pytest.mark.gpu
ULP = 2.0 ** -24 * 1.02
LEAST = 2 * 2.0 ** -149
S, P, D, FFN = 20, 2400, 1412, 1500   # neither tiles nor stages divide the widths
COUNTS = [1, 2, 3, 1, 0, 67, 129, 64] + [2133 // 12] * 12
COUNTS[-1] += P - sum(COUNTS)
OFF = np.concatenate([[0], np.cumsum(COUNTS)]).astype(np.int32)


def _normal(seed, *shape):
    return torch.randn(shape, generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV)


def _shape(act="gelu", d=D, ffn=FFN):
    return lz.Shape(P, d, ffn, S, 1, 1, S, lz.LZ_F32, lz.LZ_GELU if act == "gelu" else lz.LZ_SWIGLU)


def _up(x, w1, act="gelu"):
    """z and h of the training forward: the first GEMM's sums and their activations."""
    n1 = w1.shape[2]
    ffn, d = n1 if act == "gelu" else n1 // 2, x.shape[1]
    shape = _shape(act, d, ffn)
    off = torch.from_numpy(OFF).to(DEV)
    w2 = torch.zeros((S, ffn, d), device=DEV)
    z, h, yp = (torch.empty((P, n), device=DEV) for n in (n1, ffn, d))
    ws = torch.empty(lz.lz_train_workspace_bytes(shape), dtype=torch.uint8, device=DEV)
    lz.lz_ffn_forward_train(x, off, w1, w2, shape, z, h, yp, ws, ws.numel())
    return z, h


def _gradients(x, h, dyp, accumulate):
    """dW1 [S, D, D] and dW2 [S, D, D] where dZ is dyp: W2 the identity, gelu'(30) = 1."""
    shape = _shape("gelu", D, D)
    off = torch.from_numpy(OFF).to(DEV)
    w1, w2 = torch.zeros((S, D, D), device=DEV), torch.eye(D, device=DEV).repeat(S, 1, 1)
    z, dxp = torch.full((P, D), 30.0, device=DEV), torch.empty((P, D), device=DEV)
    dw1, dw2 = torch.zeros((S, D, D), device=DEV), torch.zeros((S, D, D), device=DEV)
    ws = torch.empty(lz.lz_train_workspace_bytes(shape), dtype=torch.uint8, device=DEV)
    call = lz.lz_ffn_backward_accumulate if accumulate else lz.lz_ffn_backward
    call(dyp, x, z, h, off, w1, w2, shape, dxp, dw1, dw2, ws, ws.numel())
    return dw1, dw2


def _rows64(x, w):
    """x [P, K] against its slots' w [S, K, n], in fp64."""
    return torch.cat([x[OFF[s]:OFF[s + 1]].double() @ w[s].double() for s in range(S)])


def _same_bits(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("accumulate", [False, True])
def test_gradients_of_slots_of_a_few_rows(accumulate):
    x, h, dyp = _normal(1, P, D), _normal(2, P, D), _normal(3, P, D)
    dw1, dw2 = _gradients(x, h, dyp, accumulate)
    for s in range(4):
        a, b = OFF[s], OFF[s + 1]
        for got, left in ((dw1, x), (dw2, h)):
            want = left[a:b].double().T @ dyp[a:b].double()
            size = left[a:b].double().abs().T @ dyp[a:b].double().abs()
            assert float(((got[s].double() - want).abs() / size).max()) <= (b - a + (b - a > 1)) * ULP, s


def test_sums_of_which_one_product_is_not_zero():
    x, w1 = torch.zeros((P, D), device=DEV), _normal(4, S, D, FFN)
    at = torch.arange(P, device=DEV) * 7 % D
    x[torch.arange(P, device=DEV), at] = _normal(5, P)
    z, _ = _up(x, w1)
    want = _rows64(x, w1)
    assert float(((z.double() - want).abs() / want.abs()).max()) <= ULP


@pytest.mark.parametrize("scale", [1e-19, 1e-33, 1e-35, 1e-37, 1e-40])
def test_small_rows_and_columns_beside_ordinary_ones(scale):
    """Single rows of x and columns of w1: each is as exact as an ordinary one, by its own largest value (at 1e-19 also where
    they meet: products of 1e-38).  A sum of 1412 products: a random walk of 44 steps of at most three roundings."""
    x, w1 = _normal(6, P, D), _normal(7, S, D, FFN)
    rows, cols = torch.arange(0, P, 5, device=DEV), torch.arange(0, FFN, 7, device=DEV)
    x[rows] *= scale
    w1[:, :, cols] *= scale
    z, _ = _up(x, w1)
    want, bound = _rows64(x, w1), 1e-6
    other_cols = torch.tensor([c for c in range(FFN) if c % 7], device=DEV)
    for part in (other_cols, cols):
        err, big = (z[:, part].double() - want[:, part]).abs(), want[:, part].abs()
        assert bool((err.amax(1) <= bound * big.amax(1) + LEAST).all())
    other_rows = torch.tensor([r for r in range(P) if r % 5], device=DEV)
    for part in (other_rows, rows):
        err, big = (z[part].double() - want[part]).abs(), want[part].abs()
        assert bool((err.amax(0) <= bound * big.amax(0) + LEAST).all())


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("scale", [1e-33, 1e-36])
def test_small_columns_of_the_gradients(scale, accumulate):
    """A column of h is a row of dW2, a column of x one of dW1, a column of dyp one of both."""
    x, h, dyp = _normal(8, P, D), _normal(9, P, D), _normal(10, P, D)
    some = torch.arange(0, D, 9, device=DEV)
    h[:, some] *= scale
    x[:, some + 3] *= scale
    dyp[:, some] *= scale
    for got, left, small in zip(_gradients(x, h, dyp, accumulate), (x, h), (some + 3, some)):
        for s in np.flatnonzero(COUNTS):
            a, b = OFF[s], OFF[s + 1]
            want = left[a:b].double().T @ dyp[a:b].double()
            size = left[a:b].double().abs().T @ dyp[a:b].double().abs()
            # of up to 180 products: three roundings in 32 k and one where the halves meet
            bound = min(b - a + (b - a > 1), 3 * (-(-(b - a) // 32)) + 1) * ULP
            assert bool(((got[s].double() - want).abs() <= bound * size + LEAST).all()), s


def _spoil(v, rows):
    """Infinities, NaNs and numbers near the largest in the given rows of v; 1e30: finite, past the split's range."""
    v = v.clone()
    v[rows[0], 7], v[rows[1], 1], v[rows[2], 9] = float("inf"), float("-inf"), float("nan")
    v[rows[3], 0], v[rows[3], 1] = float("inf"), float("-inf")
    v[rows[4]] *= 1e30
    v[rows[5]] = 3.0e38
    return v


def _check_spoiled(got, clean, want, rows, others):
    """got: one row per row of the operand; want: fp64 of a fp32 operand in which infinities stand for themselves."""
    assert _same_bits(got[others], clean[others])
    for i in (0, 1, 2, 3, 5):
        w = want[rows[i]].float()
        assert torch.equal(w.isnan(), got[rows[i]].isnan())
        assert torch.equal(w.isinf(), got[rows[i]].isinf())
        assert torch.equal(torch.sign(w[w.isinf()]), torch.sign(got[rows[i]][w.isinf()]))
    w = want[rows[4]]
    assert float((got[rows[4]].double() - w).abs().max()) <= 2e-6 * float(w.abs().max())


@pytest.mark.parametrize("act", ["gelu", "swiglu"])
@pytest.mark.parametrize("gather", [False, True])
def test_rows_past_the_splits_range_and_their_neighbours(act, gather):
    n1 = FFN * (2 if act == "swiglu" else 1)
    x, w1 = _normal(11, P, D), 0.5 + torch.rand((S, D, n1), generator=torch.Generator(device=DEV).manual_seed(12), device=DEV)
    rows = [0, 5, 40, 76, 300, 2399]
    others = torch.tensor([r for r in range(P) if r not in rows], device=DEV)
    bad = _spoil(x, rows)
    if not gather:
        (z0, h0), (z, h) = _up(x, w1, act), _up(bad, w1, act)
        _check_spoiled(z, z0, _rows64(bad, w1), rows, others)
        assert _same_bits(h[others], h0[others])
        return
    # the same bits as of the reshuffled copy, whole layer: the second GEMM's tiles meet the rows' infinities too
    shape, off = _shape(act), torch.from_numpy(OFF).to(DEV)
    w2 = _normal(13, S, FFN, D)
    perm = torch.from_numpy(np.random.default_rng(14).permutation(P).astype(np.int32)).to(DEV)
    ws = torch.empty(lz.lz_ffn_workspace_bytes(shape), dtype=torch.uint8, device=DEV)
    y = []
    for v in (x, bad):
        unpermuted = torch.empty_like(v)
        unpermuted[perm.long()] = v
        for fused in (False, True):
            y.append(torch.full((P, D), 7.0, device=DEV))
            if fused: lz.lz_expert_ffn_gather(unpermuted, perm, off, w1, w2, shape, y[-1], ws, ws.numel())
            else: lz.lz_expert_ffn(v, off, w1, w2, shape, y[-1], ws, ws.numel())
    assert _same_bits(y[0], y[1]) and _same_bits(y[2], y[3])
    assert _same_bits(y[0][others], y[2][others])
    assert y[0].isfinite().all() and not y[2][rows[0]].isfinite().any()


@pytest.mark.parametrize("accumulate", [False, True])
def test_gradients_past_the_splits_range_and_their_neighbours(accumulate):
    x, h = _normal(15, P, D), _normal(16, P, D)
    dyp = 0.5 + torch.rand((P, D), generator=torch.Generator(device=DEV).manual_seed(17), device=DEV)
    cols = [0, 5, 40, 76, 300, 1411]
    others = torch.tensor([c for c in range(D) if c not in cols], device=DEV)
    bad_h, bad_x = _spoil(h.T, cols).T.contiguous(), _spoil(x.T, cols).T.contiguous()
    for got, clean, left in zip(_gradients(bad_x, bad_h, dyp, accumulate), _gradients(x, h, dyp, accumulate), (bad_x, bad_h)):
        for s in np.flatnonzero(COUNTS):
            a, b = OFF[s], OFF[s + 1]
            _check_spoiled(got[s], clean[s], left[a:b].double().T @ dyp[a:b].double(), cols, others)
