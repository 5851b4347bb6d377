"""Which kernel a combine backward launches and how its tokens are shared out, on a host without a GPU."""
from hip_record import recorded

# T, d, k, dtype: the kernel ("elements", or "vectors" for how many choices, through the caches or past them)
CASES = [
    ((16000, 92, 1, 0), "elements"), ((16000, 96, 1, 0), "vectors 1"), ((16000, 97, 1, 0), "elements"),
    ((5448, 320, 2, 0), "vectors 2"), ((5448, 320, 3, 0), "vectors 4"), ((5448, 320, 4, 0), "vectors 4"),
    ((4096, 96, 5, 0), "vectors 8"), ((4097, 96, 5, 0), "elements"), ((4096, 92, 8, 0), "elements"),
    ((2 ** 17, 512, 1, 0), "vectors 1 past"), ((26214, 512, 2, 0), "vectors 2"), ((26215, 512, 2, 0), "vectors 2 past"),
    ((20000, 384, 4, 0), "vectors 4 past"), ((11915, 512, 5, 0), "elements"), ((11916, 512, 5, 0), "vectors 8 past"),
    ((16000, 8, 1, 1), "vectors 8 past"), ((64, 256, 2, 1), "vectors 8 past"), ((64, 260, 2, 1), "elements"),
]


def _kernel(call):
    name = call.split()[1]
    if "generic" in name:
        return "elements"
    at = name.index("Li")
    return "vectors " + name[at + 2] + (" past" if name[at + 4:].startswith("Lb1") else "")


def test_combine_backward_routes(tmp_path):
    out = recorded(tmp_path, f"""
A, out = At(1 << 20), []
for T, d, k, dtype in {[s for s, _ in CASES]}:
    s = lz.Shape(T, d, 64, 8, k, 2, 4, dtype, lz.LZ_GELU)
    rc = code(lz.lz_combine_backward, A, A, A, A, s, A, A)
    out.append((rc, calls()))
""")
    for (rc, calls), (shape, want) in zip(out, CASES):
        assert rc == 0 and len(calls) == 1 and _kernel(calls[0]) == want, (shape, calls)
        groups, threads = (int(v) for v in calls[0].split()[2:])
        assert (groups, threads) == (-(-shape[0] // 4), 256 * -(-shape[0] // 4)), shape     # four tokens of 256 threads


def test_a_whole_pass_takes_the_same_kernel(tmp_path):
    """With the tables' workgroups ahead: dgates has the bits of the call by itself.  A workgroup has eight waves, for the tables,
    and four tokens where that gives none of the 256 CUs a second workgroup."""
    cases = [(T, d, k, dtype) for (T, d, k, dtype), _ in CASES if d * k < 2000] + [(1024, 64, 2, 1), (1025, 64, 2, 1)]
    out = recorded(tmp_path, f"""
from paper_2407_04656_amd.binding import _LayerBuffers, lz_layer_backward
out = []
for T, d, k, dtype in {cases}:
    s = lz.Shape(T, d, 64, 8, k, 2, 4, dtype, lz.LZ_GELU)
    b = _LayerBuffers(**{{n: 1 << 20 for n, t in _LayerBuffers._fields_}})
    b.train_ws_bytes = lz.lz_train_workspace_bytes(s)
    rc = code(lz_layer_backward, s, b, At(1 << 20))
    out.append((rc, [c for c in calls() if "combine_backward" in c]))
""")
    wanted = dict(CASES)
    for (rc, calls), case in zip(out, cases):
        assert rc == 0 and len(calls) == 1, (case, rc, calls)
        if case in wanted:
            assert _kernel(calls[0]) == wanted[case], (case, calls)
        groups, threads = (int(v) for v in calls[0].split()[2:])
        tokens = 4 if case[0] <= 1024 else 8
        assert threads == 512 * groups and 1 <= groups - -(-case[0] // tokens) <= 5, (case, calls)
