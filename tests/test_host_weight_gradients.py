"""Which whole backward passes have both weight gradients in one launch, on a host without a GPU (256 CUs)."""
from hip_record import recorded

# T, d, ffn, E, k, N, c, dtype, act; launches of the weight gradients
CASES = [
    ((429, 3072, 3840, 8, 8, 5, 10, 1, 1), 2), ((40960, 768, 3072, 8, 1, 10, 6, 1, 0), 1),
    ((500, 2048, 3840, 8, 2, 4, 8, 1, 0), 1), ((500, 2048, 4096, 8, 2, 4, 8, 1, 0), 2),     # 7680 and 8192 tiles of 256 x 256
    ((2048, 2048, 4096, 8, 2, 4, 8, 1, 0), 1), ((2047, 2048, 4096, 8, 2, 4, 8, 1, 0), 2),   # 128 rows a slot
    ((261887, 64, 8192, 1, 1, 1, 1, 1, 0), 1), ((261888, 64, 8192, 1, 1, 1, 1, 1, 0), 2),   # an operand of 4 GiB
    ((22074, 192, 384, 5, 4, 11, 2, 0, 0), 1), ((14091, 137, 128, 60, 1, 2, 32, 0, 1), 1),  # fp32 kernel: one wave, by elements,
    ((500, 1024, 1024, 8, 2, 10, 8, 0, 0), 1), ((16000, 512, 2048, 8, 2, 13, 16, 0, 0), 1),   # four side by side, split
    ((300, 112, 128, 62, 3, 10, 11, 0, 1), 2),                                              # kernels of their own
]


def test_passes_with_both_in_one_launch(tmp_path):
    out = recorded(tmp_path, f"""
from paper_2407_04656_amd.binding import _LayerBuffers, lz_layer_backward
out = []
for case in {[s for s, _ in CASES]}:
    s = lz.Shape(*case)
    for accumulate in (0, 1):
        b = _LayerBuffers(**{{n: 1 << 20 for n, t in _LayerBuffers._fields_}})
        b.train_ws_bytes = lz.lz_train_workspace_bytes(s)
        rc = code(lz_layer_backward, s, b, At(1 << 20), bool(accumulate))
        out.append((rc, [c for c in calls() if "gemm_" in c]))
""")
    for i, (case, want) in enumerate(CASES):
        for rc, gemms in out[2 * i:2 * i + 2]:
            assert rc == 0 and len(gemms) == 2 + want, (case, rc, gemms)        # with those of dH and dxp


def test_sums_that_one_grid_cannot_hold_are_two_launches(tmp_path):
    """A grid has fewer than 2^32 threads in x, a 16-byte piece each: slots of 2^31 pieces a matrix fit one by one."""
    out = recorded(tmp_path, """
from paper_2407_04656_amd.binding import _LayerBuffers, lz_layer_backward
out = []
for d in ((1 << 17) - 64, 1 << 17):
    s = lz.Shape(1, d, 1 << 17, 1, 1, 1, 1, lz.LZ_BF16, lz.LZ_GELU)
    b = _LayerBuffers(**{n: 1 << 20 for n, t in _LayerBuffers._fields_})
    b.train_ws_bytes = lz.lz_train_workspace_bytes(s)
    rc = code(lz_layer_backward, s, b, At(1 << 20))
    out.append((rc, [int(c.split()[3]) for c in calls() if "reduce_replicas" in c]))
""")
    for (rc, threads), launches in zip(out, (1, 2)):
        assert rc == 0 and len(threads) == launches and all(n < 2 ** 32 for n in threads), (rc, threads)
