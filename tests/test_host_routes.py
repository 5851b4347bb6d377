"""Which kernels a call launches, on a host without a GPU: the rules that choose by size, alignment and place."""
from hip_record import recorded


def test_rows_past_32_bit_offsets_stay_off_the_bf16_kernels(tmp_path):
    """dZ rows of 2 ffn elements: 256 of them are 2^32 bytes from ffn = 2^22 on, one more than a descriptor holds."""
    out = recorded(tmp_path, """
A, out = At(1 << 20), []
for ffn in ((1 << 22) - 64, 1 << 22):
    s = lz.Shape(192, 64, ffn, 192, 1, 48, 4, lz.LZ_BF16, lz.LZ_SWIGLU)
    rc = code(lz.lz_ffn_backward, A, A, A, A, A, A, A, s, A, A, A, A, lz.lz_train_workspace_bytes(s))
    out.append((rc, sum("gemm_mfma" in c for c in calls())))
""")
    assert out[0] == [0, 4]    # dH, dxp and both weight gradients: 96 wide tiles in the least of them
    assert out[1] == [0, 0]


def test_transfers_of_slots_too_large_for_a_grid_are_copies(tmp_path):
    """A grid holds fewer than 2^32 threads in x; four 16-byte pieces are a thread's."""
    out = recorded(tmp_path, """
out = []
for d, ffn in ((1 << 18, (1 << 18) - 1), (1 << 18, 1 << 18)):     # 2^34 - 2^16 and 2^34 pieces of a slot's w1
    s = lz.Shape(1, d, ffn, 1, 1, 1, 1, lz.LZ_F32, lz.LZ_GELU)
    rc = code(lz.lz_apply_transfers, [(0, 0, 0, 0)], At(1 << 52), At(2 << 52), 1, At(3 << 52), At(4 << 52), 1, s)
    out.append((rc, [c.split()[0] for c in calls()]))
""")
    assert out == [[0, ["launch"]], [0, ["copy", "copy"]]]
