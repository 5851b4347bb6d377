"""Routing and dispatch at the edges of their layouts: every lane-group size, partial pieces, unaligned logits, ties,
one to 64 ranks, chunks that end anywhere.  Integer results bit for bit; gates to the fp32 bound of the layer tests."""
import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz
from oracle import moe_layer as om

from gpu_util import DEV, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E", [1, 3, 4, 5, 8, 9, 16, 17, 32, 33, 63, 64, 65, 128, 129, 255, 256])
def test_route_sizes(E):
    T = 77
    rng = np.random.default_rng(E)
    for k in sorted({1, min(2, E), min(8, E)}):
        logits = rng.standard_normal((T, E)).astype(np.float32)
        logits[::3] = np.round(logits[::3])              # many ties
        logits[5] = 0.0
        logits[6] = np.where(rng.random(E) < 0.5, -0.0, 0.0)
        logits[7] = -3.0e38
        ref_ids, ref_gates = om.route(logits, k)
        for shift in (0, 1):                              # 16-byte aligned, then not
            buf = torch.zeros(T * E + 4, dtype=torch.float32, device=DEV)
            view = buf[shift:shift + T * E].view(T, E)
            view.copy_(to_dev(logits))
            ids = torch.empty((T, k), dtype=torch.int32, device=DEV)
            gates = torch.empty((T, k), dtype=torch.float32, device=DEV)
            lz.lz_route(view, T, E, k, ids, gates)
            assert np.array_equal(to_host(ids), ref_ids)
            assert np.max(np.abs(to_host(gates) - ref_gates) / ref_gates) <= 2e-6


@pytest.mark.parametrize("T,E,k,N,c", [(1, 1, 1, 1, 1), (129, 3, 2, 2, 2), (1000, 17, 5, 3, 6), (2000, 256, 8, 64, 5),
                                       (4097, 130, 3, 33, 4), (640, 8, 1, 5, 64), (3000, 64, 6, 17, 4),
                                       # one workgroup for all, at and past its bounds: pairs, triples, slots, experts
                                       (4096, 8, 1, 16, 8), (4097, 8, 1, 16, 8), (512, 2, 2, 32, 16), (100, 2, 2, 33, 15),
                                       (50, 32, 8, 8, 64), (40, 33, 3, 4, 9), (1, 32, 1, 1, 40)])
def test_dispatch_sizes(T, E, k, N, c):
    rng = np.random.default_rng(T + E)
    logits = (rng.standard_normal((T, E)) - 1.1 * np.log(1.0 + rng.permutation(E))).astype(np.float32)
    ids, _ = om.route(logits, k)
    plan = np.concatenate([np.arange(E), rng.integers(0, E, size=N * c - E)]).astype(np.int32)
    rng.shuffle(plan)
    cuts = np.sort(rng.integers(0, T + 1, size=N - 1))    # ragged ranks, some of them empty
    off = np.concatenate([[0], cuts, [T]]).astype(np.int32)
    ref = om.plan_dispatch(ids, off, plan, E, N, c)
    layer = lz.MoELayer(lz.Shape(T, 8, 8, E, k, N, c, lz.LZ_F32, lz.LZ_GELU), DEV)
    layer.set_plan(plan, off)
    layer.route(to_dev(logits))
    layer.plan_dispatch()
    assert int(layer.status.item()) == 0
    for name in ("Tej", "D", "slot_counts", "slot_offsets", "pair_to_row", "row_to_pair"):
        assert np.array_equal(to_host(getattr(layer, name)), ref[name]), name
