"""The dispatcher's three sequences of kernels at the edges of the rules that choose between them (test_host_dispatch_route.py
holds those to these sizes), and of their chunks and tables.  Integer results bit for bit."""
import numpy as np
import pytest
import torch

import paper_2407_04656_amd as lz
from oracle import moe_layer as om

from gpu_util import DEV, to_dev, to_host
from test_gpu_dispatch_sizes import test_dispatch_sizes as check_sizes
from test_gpu_parity import test_plan_dispatch_is_deterministic_and_flags_bad_input as check_flags

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,k,N,c", [
    (1024, 24, 2, 8, 4), (1025, 24, 2, 8, 4), (1024, 25, 2, 8, 4),     # one workgroup, and past it by a pair and an expert
    (4096, 33, 2, 8, 5), (4097, 33, 2, 8, 5), (8192, 9, 1, 64, 1),     # counted by the experts' workgroups, by a launch
    (1024, 30, 1, 1, 40), (1025, 30, 1, 1, 40), (1151, 30, 1, 2, 20),  # whole and broken groups of 8 chunks
    (3000, 256, 3, 32, 9), (3000, 256, 3, 33, 9),                      # a rank's table in LDS, and too large for it
    (70000, 12, 2, 3, 5),                                              # several workgroups a rank
])
def test_edges(T, E, k, N, c):
    check_sizes(T, E, k, N, c)


def test_flags_with_a_launch_that_counts():
    check_flags(9000)


@pytest.mark.parametrize("E", [3, 6, 8, 13, 31, 64, 129, 255, 256])
def test_every_number_of_choices(E):
    """Ties at every depth: logits of few values, all equal, both zeros; more choices than a lane holds logits."""
    rng = np.random.default_rng(E)
    T = 131
    logits = rng.integers(-2, 3, size=(T, E)).astype(np.float32) * np.float32(0.25)
    logits[::2] += rng.standard_normal((len(logits[::2]), E)).astype(np.float32)
    logits[3] = 1.0
    logits[4] = np.where(rng.random(E) < 0.5, -0.0, 0.0)
    logits[5] = np.float32(-3.4e38)
    logits[6, E - 1] = np.float32(3.4e38)
    for k in range(1, min(E, 8) + 1):
        ref_ids, ref_gates = om.route(logits, k)
        ids = torch.empty((T, k), dtype=torch.int32, device=DEV)
        gates = torch.empty((T, k), dtype=torch.float32, device=DEV)
        lz.lz_route(to_dev(logits), T, E, k, ids, gates)
        assert np.array_equal(to_host(ids), ref_ids), k
        bound = 2e-6 * ref_gates + 1e-37       # the fp32 bound of the layer tests, and gates below the least normal number
        assert np.all(np.abs(to_host(gates) - ref_gates) <= bound), k
