"""When a layer's pass is one call and when it keeps to its steps, on a host without a GPU."""
import pytest

from hip_record import recorded

LAYER = """
import torch
from paper_2407_04656_amd import binding
binding._stream = lambda: 0
def aligned(n):
    t = torch.zeros(n + 256, dtype=torch.uint8)
    return t[-t.data_ptr() % 256:][:n]
def layer_of(cls=lz.MoELayer):
    l = cls(lz.Shape(64, 64, 64, 8, 2, 4, 4, lz.LZ_BF16, lz.LZ_GELU), "cpu")
    l.set_plan([s % 8 for s in range(16)], [0, 16, 32, 48, 64])
    l.set_slot_weights(*(torch.zeros(16, 64, 64, dtype=l.xp.dtype) for _ in range(2)))
    l.enable_training()
    l.enable_accumulation()
    l.plan_ws, l.ffn_ws, l.train_ws = (aligned(n) for n in (l.plan_ws_bytes, l.ffn_ws_bytes, l.train_ws_bytes))
    return l
x = torch.zeros(64, 64, dtype=torch.bfloat16)
logits = torch.zeros(64, 8)
"""
STEPS = ["route", "plan_dispatch", "permute", "expert_ffn", "unpermute_combine"]


@pytest.mark.parametrize("place", ["class", "subclass", "object"])
def test_a_step_of_its_own_is_taken(tmp_path, place):
    out = recorded(tmp_path, LAYER + f"""
out = []
for step in {STEPS}:
    seen, original = [], getattr(lz.MoELayer, step)
    def own(self, *args):
        seen.append(1)
        return original(self, *args)
    l = layer_of(type("Timed", (lz.MoELayer,), dict([(step, own)])) if {place!r} == "subclass" else lz.MoELayer)
    if {place!r} == "object": setattr(l, step, lambda *args: own(l, *args))
    if {place!r} == "class": setattr(lz.MoELayer, step, own)
    counts = []
    for run in (l.forward, l.forward_fused, l.forward_train):
        run(logits, x)
        counts.append(len(seen))
    if {place!r} == "class": setattr(lz.MoELayer, step, original)       # one call again
    calls()
    layer_of().forward(logits, x)
    out.append((counts, len(calls())))
""")
    for step, (counts, launches) in zip(STEPS, out):
        fused = step not in ("permute", "expert_ffn")       # which that pass does without
        train = step != "expert_ffn"
        assert counts == [1, 1 + fused, 1 + fused + train], step
        assert launches == 5        # routing and tables in the dispatcher's launch


def test_a_pass_asks_for_its_own_buffers_only(tmp_path):
    """xp is not used by a fused forward, ffn_ws by no training step, the plan's other buffers by no backward."""
    out = recorded(tmp_path, LAYER + """
out = []
def without(names, *passes):
    l = layer_of()
    l.forward_train(logits, x)
    for n in names:
        delattr(l, n)
    for name, *args in passes:
        calls()
        getattr(l, name)(*args)
        out.append(len(calls()))
without(["xp", "train_ws", "z", "h"], ("forward_fused", logits, x))
without(["train_ws", "z", "h", "dyp", "dw1_slot"], ("forward", logits, x))
without(["ffn_ws"], ("forward_train", logits, x))
without(["ffn_ws", "plan_ws", "row_to_pair", "slot_counts", "Tej", "D", "status", "y", "dw1_acc"], ("backward", x))
without(["ffn_ws", "plan_ws", "dw1", "dw1_slot"], ("backward_accumulate", x))
""")
    assert all(out) and len(out) == 5
