"""Slot transfers of a re-plan against the same copies on the host: every source and slot count of a launch's list,
partial blocks, and the lists that must keep their order (repeated destinations, one buffer for old and new)."""
import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz

from gpu_util import DEV, to_dev, to_host

pytestmark = pytest.mark.gpu


def _apply(xfers, w1, w2, S_old, n1, n2, S_new, shape):
    lz.lz_apply_transfers([(d, s, 0, 0) for d, s in xfers], w1, w2, S_old, n1, n2, S_new, shape)
    torch.cuda.synchronize()


@pytest.mark.parametrize("d,ffn,S_old,S_new,dtype", [
    (4, 4, 3, 5, lz.LZ_F32),          # one block of two pieces
    (64, 72, 40, 300, lz.LZ_BF16),    # more slots than one launch lists
    (8, 16, 300, 200, lz.LZ_BF16),    # more sources than one launch lists
    (128, 260, 7, 9, lz.LZ_F32),      # blocks that end inside a slot
    (5, 3, 4, 6, lz.LZ_BF16),         # slots of no whole 16-byte pieces
])
def test_transfers(d, ffn, S_old, S_new, dtype):
    rng = np.random.default_rng(d * ffn)
    shape = lz.Shape(1, d, ffn, 1, 1, 1, 1, dtype, lz.LZ_SWIGLU)
    dt = np.float32 if dtype == lz.LZ_F32 else np.uint16
    old = [rng.integers(0, 1000, size=(S_old, *sh)).astype(dt) for sh in ((d, 2 * ffn), (ffn, d))]
    new = [rng.integers(0, 1000, size=(S_new, *sh)).astype(dt) for sh in ((d, 2 * ffn), (ffn, d))]
    dsts = rng.permutation(S_new)[:S_new - 1]             # one slot keeps what it holds
    xfers = [(int(t), int(rng.integers(0, S_old))) for t in dsts]
    for repeated in (False, True):
        if repeated:
            xfers += [(xfers[0][0], (xfers[0][1] + 1) % S_old)]   # a destination twice: the last one counts
        dev_old, dev_new = [to_dev(a) for a in old], [to_dev(a) for a in new]
        _apply(xfers, *dev_old, S_old, *dev_new, S_new, shape)
        for o, n, got in zip(old, new, dev_new):
            ref = n.copy()
            for t, s in xfers:
                ref[t] = o[s]
            assert np.array_equal(to_host(got), ref)


def test_transfers_inside_one_buffer_follow_the_list():
    shape = lz.Shape(1, 8, 8, 1, 1, 1, 1, lz.LZ_F32, lz.LZ_GELU)
    w1, w2 = (np.random.default_rng(s).standard_normal((4, 8, 8)).astype(np.float32) for s in (1, 2))
    a, b = to_dev(w1), to_dev(w2)
    xfers = [(1, 0), (2, 1), (0, 3)]
    _apply(xfers, a, b, 4, a, b, 4, shape)
    for t, s in xfers:
        w1[t], w2[t] = w1[s], w2[s]
    assert np.array_equal(to_host(a), w1) and np.array_equal(to_host(b), w2)


def test_transfers_under_capture():
    """The one-kernel form is taken, captured and replayed like the other calls of a pass."""
    shape = lz.Shape(1, 64, 64, 1, 1, 1, 1, lz.LZ_BF16, lz.LZ_GELU)
    w1, w2 = (torch.randn((3, 64, 64), device=DEV).bfloat16() for _ in range(2))
    n1, n2 = (torch.zeros((4, 64, 64), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    xfers = [(0, 2, 0, 0), (3, 2, 0, 0), (1, 0, 0, 0)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lz.lz_apply_transfers(xfers, w1, w2, 3, n1, n2, 4, shape)
    for replay in range(3):
        w1.add_(replay)
        n1.zero_(), n2.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for old, new in ((w1, n1), (w2, n2)):
            for t, s, _, _ in xfers:
                assert torch.equal(new[t], old[s])
            assert not new[2].any()
