"""Routing at both sides of the line between its two ways of selecting, rows that are no 16-byte pieces: ids bit for bit, gates
within the fp32 bound of the layer tests."""
import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz
from oracle import moe_layer as om

from gpu_util import DEV, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [4096, 4097, 12289])
@pytest.mark.parametrize("E,k", [(65, 5), (81, 6), (127, 7)])
def test_both_sides(T, E, k):
    rng = np.random.default_rng(T + E)
    logits = rng.integers(-2, 3, size=(T, E)).astype(np.float32) * np.float32(0.25)        # ties at every depth
    logits[::2] += rng.standard_normal((len(logits[::2]), E)).astype(np.float32)
    ref_ids, ref_gates = om.route(logits, k)
    ids = torch.empty((T, k), dtype=torch.int32, device=DEV)
    gates = torch.empty((T, k), dtype=torch.float32, device=DEV)
    lz.lz_route(to_dev(logits), T, E, k, ids, gates)
    assert np.array_equal(to_host(ids), ref_ids)
    assert np.all(np.abs(to_host(gates) - ref_gates) <= 2e-6 * ref_gates + 1e-37)
