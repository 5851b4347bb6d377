"""The combine backward's kernels at both sides of the rules between them (test_host_combine_backward.py), against 64 bits."""
import pytest
import torch

import paper_2407_04656_amd as lz

from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,k,dtype", [
    (4097, 92, 1, lz.LZ_F32), (4097, 96, 1, lz.LZ_F32), (5, 260, 2, lz.LZ_F32), (131, 516, 3, lz.LZ_F32), (131, 100, 4, lz.LZ_F32),
    (4096, 96, 5, lz.LZ_F32), (4097, 96, 5, lz.LZ_F32), (1, 1028, 8, lz.LZ_F32), (26215, 512, 2, lz.LZ_F32),
    (2 ** 17 // 4, 1024, 1, lz.LZ_F32), (12000, 512, 8, lz.LZ_F32), (131, 264, 8, lz.LZ_BF16), (131, 97, 3, lz.LZ_BF16),
])
def test_against_64_bits(T, d, k, dtype):
    g = torch.Generator(device=DEV)
    g.manual_seed(T + d)
    tdt = torch.float32 if dtype == lz.LZ_F32 else torch.bfloat16
    dy, yp = (torch.randn((n, d), generator=g, device=DEV).to(tdt) for n in (T, T * k))
    gates = torch.rand((T, k), generator=g, device=DEV)
    rows = torch.randperm(T * k, generator=g, device=DEV).to(torch.int32)
    dropped = torch.zeros(T * k, dtype=torch.bool, device=DEV)
    dropped[::7] = True             # pairs without a row: no gradient of theirs is written
    row_of = torch.where(dropped, -1, rows).contiguous()
    dyp = torch.full((T * k, d), 3.0, dtype=tdt, device=DEV)
    dgates = torch.full((T, k), 3.0, device=DEV)
    lz.lz_combine_backward(dy, yp, row_of, gates, lz.Shape(T, d, 64, 8, k, 1, 8, dtype, lz.LZ_GELU), dyp, dgates)
    for t0 in range(0, T, 4096):    # in pieces: the 64-bit rows of the large cases
        sel = slice(t0 * k, (t0 + 4096) * k)
        r, lost = rows[sel].long(), dropped[sel]
        y64, yp64 = dy[t0:t0 + 4096].double().repeat_interleave(k, 0), yp[r].double()
        want = (y64 * yp64).sum(1)
        # fp32 sums of d products: a lane's one after the other, whole 16-byte pieces of them, and six steps of the wave, each
        # off by 2^-24 at most
        bar = (8 * -(-d // 512) + 7) * 2.0 ** -24 * (y64 * yp64).abs().sum(1)
        got = dgates.reshape(-1)[sel].double()
        assert torch.all((got - torch.where(lost, 0.0, want)).abs() <= bar)
        exact = gates.reshape(-1)[sel].double()[:, None] * y64      # one rounding to fp32, one to the tensor's type
        step = 2.0 ** -23 if dtype == lz.LZ_F32 else 2.0 ** -8
        wrote = dyp[r].double()
        assert torch.all(torch.where(lost[:, None], wrote == 3.0, (wrote - exact).abs() <= step * exact.abs()))
