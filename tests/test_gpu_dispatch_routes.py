"""The dispatcher's three sequences of kernels at the edges of the rules that choose between them (test_host_dispatch_route.py
holds those to these sizes), and of their chunks and tables.  Integer results bit for bit."""
import pytest

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
