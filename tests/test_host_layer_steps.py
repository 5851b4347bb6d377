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


def test_a_refusal_names_its_step(tmp_path):
    out = recorded(tmp_path, LAYER + """
out = []
def refused(name, change, *args):
    l = layer_of()
    if change: setattr(l, *change)
    try:
        getattr(l, name)(*args)
    except lz.LzError as e:
        out.append((str(e).split(":")[0], e.code))
    else:
        out.append(None)
big = lz.Shape(64, 64, 64, 8, 9, 4, 4, lz.LZ_BF16, lz.LZ_GELU)
for name in ("forward", "forward_fused", "forward_train"):
    refused(name, None, None, x)
    refused(name, ("slot_expert", None), logits, x)
    refused(name, ("plan_ws_bytes", 64), logits, x)
    refused(name, None, logits, None)
    refused(name, ("train_ws_bytes" if name == "forward_train" else "ffn_ws_bytes", 64), logits, x)
    refused(name, ("w1", None), logits, x)
    refused(name, ("y", None), logits, x)
    refused(name, ("shape", big), logits, x)
for name in ("backward", "backward_accumulate"):
    refused(name, None, None)
    refused(name, ("w1", None), x)
    refused(name, ("train_ws_bytes", 64), x)
    refused(name, ("dx", None), x)
    refused(name, ("dlogits", None), x)
refused("backward", ("dw1", None), x)
from paper_2407_04656_amd import binding
out.append((binding.lib.lz_layer_forward(layer_of().shape._arg(), None, 64, 64, 0, 0), binding.lib.lz_layer_refused().decode()))
""")
    EINVAL, ESHAPE, EWORKSPACE = -1, -2, -3
    want = []
    for ffn in ("lz_expert_ffn", "lz_expert_ffn_gather", "lz_ffn_forward_train"):
        want += [("lz_route", EINVAL), ("lz_plan_dispatch", EINVAL), ("lz_plan_dispatch", EWORKSPACE),
                 (ffn if ffn.endswith("gather") else "lz_permute_scatter", EINVAL), (ffn, EWORKSPACE), (ffn, EINVAL),
                 ("lz_unpermute_combine", EINVAL), ("lz_route", ESHAPE)]
    for ffn in ("lz_ffn_backward", "lz_ffn_backward_accumulate"):
        want += [("lz_combine_backward", EINVAL), (ffn, EINVAL), (ffn, EWORKSPACE), ("lz_permute_backward", EINVAL),
                 ("lz_route_backward", EINVAL)]
    want += [("lz_reduce_replica_grads_dtype", EINVAL), (EINVAL, "lz_layer_forward")]
    assert [tuple(o) for o in out] == want


def test_a_call_is_refused_before_the_device_is_asked_for():
    """Bad arguments are that on a host without a GPU too, as the calls by themselves have it."""
    import paper_2407_04656_amd as lz
    from paper_2407_04656_amd import binding

    class At:
        def __init__(self, address): self.address = address
        def data_ptr(self): return self.address
        def is_contiguous(self): return True
    fields = {n: 1 << 20 for n, _ in binding._LayerBuffers._fields_}
    for k, missing, want in ((9, None, -2), (2, "yp", -1), (2, "dgates", -1)):
        shape = lz.Shape(64, 64, 64, 8, k, 4, 4, lz.LZ_BF16, lz.LZ_GELU)
        buffers = binding._LayerBuffers(**{n: v for n, v in fields.items() if n != missing})
        buffers.train_ws_bytes = lz.lz_train_workspace_bytes(shape)
        with pytest.raises(lz.LzError) as e:
            binding.lz_layer_backward(shape, buffers, At(1 << 20), stream=0)
        assert (e.value.code, str(e.value).split(":")[0]) == (want, "lz_combine_backward")
