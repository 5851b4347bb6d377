"""Accumulated weight gradients of slots without rows: the wide bf16 kernel gets no tiles for them, so their sums keep
every bit; the other slots' sums grow by their gradients, whichever slots are empty, also all of them."""
import pytest
import torch

import paper_2407_04656_amd as lz

from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts", [(0, 1, 0, 0, 70, 0), (33, 0, 0, 0, 0, 0), (0, 0, 0, 0, 0, 257), (0, 0, 0, 0, 0, 0), (5, 64, 300, 1, 65, 9)])
@pytest.mark.parametrize("d,ffn", [(256, 512), (264, 328)])
def test_sums_of_empty_slots_stay_as_they_are(counts, d, ffn):
    S, rows = len(counts), sum(counts)
    P = max(rows, 8)                       # with no row in any slot the batch's rows belong to none
    shape = lz.Shape(P, d, ffn, S, 1, 1, S, lz.LZ_BF16, lz.LZ_GELU)
    gen = torch.Generator(device=DEV).manual_seed(rows)
    normal = lambda *s: torch.randn(s, generator=gen, device=DEV)  # noqa: E731
    x, dyp, z, h = (normal(P, n).bfloat16() for n in (d, d, ffn, ffn))
    w1, w2 = 0.05 * normal(S, d, ffn).bfloat16(), 0.05 * normal(S, ffn, d).bfloat16()
    off = torch.tensor([sum(counts[:s]) for s in range(S + 1)], dtype=torch.int32, device=DEV)
    acc1, acc2 = normal(S, d, ffn), normal(S, ffn, d)
    acc1[:, 0, 0] = -0.0
    old1, old2 = acc1.clone(), acc2.clone()
    dxp = torch.zeros_like(x)
    ws = torch.empty(lz.lz_train_workspace_bytes(shape), dtype=torch.uint8, device=DEV)
    lz.lz_ffn_backward_accumulate(dyp, x, z, h, off, w1, w2, shape, dxp, acc1, acc2, ws, ws.numel())
    a = 0
    for s, n in enumerate(counts):
        if n == 0:
            assert torch.equal(acc1[s].view(torch.int32), old1[s].view(torch.int32))
            assert torch.equal(acc2[s].view(torch.int32), old2[s].view(torch.int32))
        else:
            zs = z[a:a + n].double().requires_grad_(True)
            torch.nn.functional.gelu(zs).backward(dyp[a:a + n].double() @ w2[s].double().T)
            for acc, old, grad in ((acc1, old1, x[a:a + n].double().T @ zs.grad), (acc2, old2, h[a:a + n].double().T @ dyp[a:a + n].double())):
                # dH and dZ are rounded to bf16 (2^-9 each) before the fp32 sums
                assert float((acc[s].double() - old[s].double() - grad).abs().max()) <= 2e-2 * float(grad.abs().max())
        a += n
