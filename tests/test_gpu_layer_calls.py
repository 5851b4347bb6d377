"""A layer's passes in one call: the bits of the single calls in every buffer, and their refusals."""
import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz

from gpu_util import DEV

pytestmark = pytest.mark.gpu

FORWARD = ("topk_ids", "topk_gates", "slot_counts", "slot_offsets", "pair_to_row", "row_to_pair", "Tej", "D", "status", "xp", "y")
BACKWARD = ("z", "h", "dyp", "dxp", "dx", "dgates", "dlogits")


class SingleCalls(lz.MoELayer):
    """The same passes, call by call."""

    def route(self, logits):
        super().route(logits)

    def backward(self, dy, accumulate=False):
        s, ws = self.shape, (self.train_ws, self.train_ws_bytes)
        lz.lz_combine_backward(dy, self.yp, self.pair_to_row, self.topk_gates, s, self.dyp, self.dgates)
        call, dw1, dw2 = ((lz.lz_ffn_backward_accumulate, self.dw1_acc, self.dw2_acc) if accumulate else
                          (lz.lz_ffn_backward, self.dw1_slot, self.dw2_slot))
        call(self.dyp, self.xp, self.z, self.h, self.slot_offsets, self.w1, self.w2, s, self.dxp, dw1, dw2, *ws)
        lz.lz_permute_backward(self.dxp, self.pair_to_row, s, self.dx)
        lz.lz_route_backward(self.dgates, self.topk_gates, self.topk_ids, s, self.dlogits)
        if not accumulate:
            for slots, out in ((self.dw1_slot, self.dw1), (self.dw2_slot, self.dw2)):
                lz.lz_reduce_replica_grads_dtype(slots, self.slot_expert, s.S, s.E, slots[0].numel(), s.dtype, out)
        return self.dx

    def backward_accumulate(self, dy):
        return self.backward(dy, True)


def _pair(T, d, ffn, E, k, N, c, dtype, act, seed=0):
    """Two layers of one shape, plan and weights, one pass by pass, one call by call; and a batch."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed + T)
    rng = np.random.default_rng(seed + T)
    shape = lz.Shape(T, d, ffn, E, k, N, c, dtype, act)
    tdt = torch.float32 if dtype == lz.LZ_F32 else torch.bfloat16
    plan = np.concatenate([np.arange(E), rng.integers(0, E, size=N * c - E)]).astype(np.int32)
    rng.shuffle(plan)
    off = np.concatenate([[0], np.sort(rng.integers(0, T + 1, size=N - 1)), [T]]).astype(np.int32)

    def normal(*size):
        return torch.randn(size, generator=gen, device=DEV).to(tdt)
    w1, w2 = 0.05 * normal(N * c, d, ffn * (2 if act == lz.LZ_SWIGLU else 1)), 0.05 * normal(N * c, ffn, d)
    layers = [cls(shape, DEV) for cls in (lz.MoELayer, SingleCalls)]
    for layer in layers:
        layer.set_plan(plan, off)
        layer.set_slot_weights(w1, w2)
        layer.enable_training()
        layer.enable_accumulation()
        for name in FORWARD + ("yp",) + BACKWARD:       # what neither writes compares equal
            getattr(layer, name).view(torch.uint8).fill_(0x11)
    logits = torch.randn((T, E), generator=gen, device=DEV)
    return layers, logits, normal(T, d), normal(T, d)


def _same(a, b, names):
    for name in names:
        x, y = getattr(a, name), getattr(b, name)
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), name


CASES = [
    (1, 64, 64, 2, 1, 1, 3, lz.LZ_BF16, lz.LZ_GELU),
    (256, 128, 256, 8, 2, 4, 4, lz.LZ_F32, lz.LZ_GELU),          # routed, planned and tabled by one workgroup
    (300, 96, 200, 3, 1, 2, 3, lz.LZ_BF16, lz.LZ_SWIGLU),
    (170, 264, 136, 16, 5, 3, 7, lz.LZ_BF16, lz.LZ_GELU),
    (64, 40, 72, 24, 3, 8, 32, lz.LZ_BF16, lz.LZ_SWIGLU),
    (70, 33, 50, 24, 3, 5, 6, lz.LZ_F32, lz.LZ_SWIGLU),
    (2048, 64, 64, 8, 1, 3, 4, lz.LZ_BF16, lz.LZ_GELU),          # planned by one workgroup, routed before
    (1500, 512, 1024, 8, 2, 4, 3, lz.LZ_F32, lz.LZ_GELU),        # the split fp32 kernel's table too
    (1500, 512, 768, 12, 4, 4, 4, lz.LZ_BF16, lz.LZ_SWIGLU),     # tables beside the placing workgroups
    (3000, 72, 130, 40, 3, 16, 64, lz.LZ_BF16, lz.LZ_GELU),      # 1024 slots, rows of no whole pieces
    (9000, 256, 512, 6, 2, 3, 4, lz.LZ_BF16, lz.LZ_GELU),
    (5000, 768, 1088, 16, 2, 8, 8, lz.LZ_BF16, lz.LZ_GELU),      # both weight gradients in one launch: several rounds,
    (400, 264, 328, 20, 2, 5, 5, lz.LZ_BF16, lz.LZ_SWIGLU),      # one round, lists of unlike lengths
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "T%d_d%d_f%d_E%d_k%d_N%d_c%d_%s%s" % (*c[:7], "fb"[c[7]], "gs"[c[8]]))
def test_passes_have_the_bits_of_the_single_calls(case):
    (one, single), logits, x, dy = _pair(*case)
    for _ in range(2):      # tables and counters of a pass before do not matter
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


def test_refusals_are_those_of_the_single_calls():
    (one, _), logits, x, dy = _pair(64, 64, 64, 8, 2, 4, 4, lz.LZ_BF16, lz.LZ_GELU)
    s = one.shape
    code = lambda f, *a: getattr(pytest.raises(lz.LzError, f, *a).value, "code")
    EINVAL, ESHAPE, EWORKSPACE = -1, -2, -3
    assert code(one.forward, None, x) == EINVAL
    assert code(one.forward, logits, None) == EINVAL
    assert code(one.forward_fused, logits, None) == EINVAL
    assert code(one.forward_train, logits, None) == EINVAL
    assert code(one.backward, None) == EINVAL
    for attribute, passes in (("w1", (one.forward, one.forward_fused, one.forward_train)), ("slot_expert", (one.forward,))):
        kept = getattr(one, attribute)
        setattr(one, attribute, None)
        for run in passes:
            assert code(run, logits, x) == EINVAL
        setattr(one, attribute, kept)
    for attribute, run in (("plan_ws_bytes", one.forward), ("ffn_ws_bytes", one.forward), ("train_ws_bytes", one.forward_train)):
        setattr(one, attribute, getattr(one, attribute) - 1)
        assert code(run, logits, x) == EWORKSPACE
        setattr(one, attribute, getattr(one, attribute) + 1)
    one.shape = lz.Shape(64, 64, 64, 8, 9, 4, 4, lz.LZ_BF16, lz.LZ_GELU)
    assert code(one.forward, logits, x) == ESHAPE
    one.shape = s
    one.forward(logits, x)
    assert int(one.status.item()) == 0


def test_a_layer_with_a_step_of_its_own_keeps_to_it():
    (one, single), logits, x, _ = _pair(64, 64, 64, 8, 2, 4, 4, lz.LZ_BF16, lz.LZ_GELU)
    calls = []
    one.permute = lambda t: (calls.append("permute"), lz.MoELayer.permute(one, t))
    one.forward(logits, x)
    single.forward(logits, x)
    assert calls == ["permute"]
    _same(one, single, FORWARD)
