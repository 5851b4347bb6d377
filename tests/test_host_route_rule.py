"""Which of its two ways of selecting a routing call takes, on a host without a GPU."""
from hip_record import recorded

# T, E, k, address of the logits: by rounds, or by sorted keys
CASES = [
    ((100000, 80, 4, 1 << 20), "rounds"), ((100000, 80, 5, 1 << 20), "sorted"), ((100000, 80, 5, (1 << 20) + 4), "rounds"),
    ((4096, 81, 5, 1 << 20), "sorted"), ((4097, 81, 5, 1 << 20), "rounds"),
    ((8192, 65, 6, 1 << 20), "sorted"), ((8193, 65, 6, 1 << 20), "rounds"),
    ((12288, 127, 7, 1 << 20), "sorted"), ((12289, 127, 7, 1 << 20), "rounds"),
    ((16384, 127, 8, 1 << 20), "sorted"), ((16385, 127, 8, 1 << 20), "rounds"),
    ((100000, 63, 5, 1 << 20), "sorted"), ((100000, 129, 5, 1 << 20), "sorted"),
]


def test_the_line_between_rounds_and_sorted_keys(tmp_path):
    out = recorded(tmp_path, f"""
out = []
for T, E, k, logits in {[s for s, _ in CASES]}:
    rc = code(lz.lz_route, At(logits), T, E, k, At(1 << 24), At(1 << 25))
    out.append((rc, calls()))
""")
    for (rc, calls), (case, want) in zip(out, CASES):
        assert rc == 0 and len(calls) == 1, (case, calls)
        name = calls[0].split()[1]                      # ...<G, V, VEC, SORTED>
        assert ("Lb1EEEv" in name) == (want == "sorted"), (case, name)
