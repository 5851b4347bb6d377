"""Which kernels a dispatch launches, on a host without a GPU."""
from hip_record import recorded

SMALL, DIRECT, TABLES = ["plan_small"], ["schedule_expert", "place"], ["count", "schedule_expert", "place"]


def test_dispatch_routes(tmp_path):
    shapes = [((1024, 24, 2, 8, 4), SMALL), ((1025, 24, 2, 8, 4), DIRECT), ((1024, 25, 2, 8, 4), DIRECT), ((0, 8, 2, 8, 4), DIRECT),
              ((4096, 33, 2, 8, 5), DIRECT), ((4097, 33, 2, 8, 5), TABLES), ((9000, 16, 2, 4, 4), TABLES)]
    out = recorded(tmp_path, f"""
A, out = At(1 << 20), []
for T, E, k, N, c in {[s for s, _ in shapes]}:
    s = lz.Shape(T, 64, 64, E, k, N, c, lz.LZ_BF16, lz.LZ_GELU)
    rc = code(lz.lz_plan_dispatch, A, s, A, A, A, A, A, A, A, A, A, A, lz.lz_plan_workspace_bytes(s))
    out.append((rc, calls()))
""")
    for (rc, calls), (shape, want) in zip(out, shapes):
        assert rc == 0 and len(calls) == len(want), shape
        assert all(name + "_kernel" in call for name, call in zip(want, calls)), (shape, calls)
