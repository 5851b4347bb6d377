"""Which kernels a call launches, on a host without a GPU: the rules that choose by size, alignment and place."""
import pytest

import paper_2407_04656_amd as lz

from hip_record import recorded


def test_rows_past_32_bit_offsets_stay_off_the_bf16_kernels(tmp_path):
    """dZ rows of 2 ffn elements: 256 of them are 2^32 bytes from ffn = 2^22 on, one more than a descriptor holds."""
    out = recorded(tmp_path, """
A, out = At(1 << 20), []
for ffn in ((1 << 22) - 64, 1 << 22):
    s = lz.Shape(192, 64, ffn, 192, 1, 48, 4, lz.LZ_BF16, lz.LZ_SWIGLU)
    rc = code(lz.lz_ffn_backward, A, A, A, A, A, A, A, s, A, A, A, A, lz.lz_train_workspace_bytes(s))
    out.append((rc, sum("gemm_mfma" in c or "gemm_narrow" in c for c in calls())))
""")
    assert out[0] == [0, 4]    # dH, dxp and both weight gradients
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


def test_transfers_between_places_are_copies(tmp_path):
    """The kernel serves buffers of the stream's own GPU; a buffer of another one, or memory the runtime does not know
    as a GPU's, is left to the runtime's copies, one per matrix and transfer, in the order of the list."""
    out = recorded(tmp_path, """
s = lz.Shape(64, 64, 64, 4, 2, 2, 2, lz.LZ_BF16, lz.LZ_GELU)
size = 64 * 64 * 2
def run(addresses, stream=0):
    rc = code(lz.lz_apply_transfers, [(0, 1, 0, 0), (2, 0, 0, 0)], At(addresses[0]), At(addresses[1]), 4,
              At(addresses[2]), At(addresses[3]), 4, s, stream=stream)
    return rc, calls()
here = [1 << 20, 2 << 20, 3 << 20, 4 << 20]
out = [run(here), run([a + (1 << 40) for a in here], stream=1), run(here, stream=1)]
for i in range(4):
    for bit in (40, 44):
        out.append(run([a + (1 << bit) * (j == i) for j, a in enumerate(here)]))
w = [here[0], here[1], here[2], here[3] + (1 << 40)]
out = [[rc, [c.split()[0] for c in cs]] for rc, cs in out] + [[[w[2 + m] + d * size, w[m] + q * size, size] for d, q in ((0, 1), (2, 0)) for m in range(2)],
       [[int(v) for v in c.split()[1:]] for c in run(w)[1]]]
""")
    for one_device in out[:2]:
        assert one_device == [0, ["launch"]]
    for across in out[2:-2]:
        assert across == [0, ["copy"] * 4]
    assert out[-1] == out[-2]


@pytest.mark.parametrize("d,ffn,k,N,c", [
    (512, 512, 1, 32, 40), (256, 128, 1, 64, 64), (4096, 14336, 2, 8, 2), (1000, 2664, 2, 6, 2), (72, 200, 1, 64, 64),
    (20000, 20000, 1, 64, 64),     # 2 GiB of x at 53687 tokens, where the fp32 kernel takes over
    (71, 205, 2, 4, 4),
])
@pytest.mark.parametrize("act", [lz.LZ_GELU, lz.LZ_SWIGLU])
@pytest.mark.parametrize("dtype", [lz.LZ_F32, lz.LZ_BF16])
def test_a_workspace_of_the_largest_batch_serves_the_smaller_ones(dtype, act, d, ffn, k, N, c):
    def sizes(T):
        s = lz.Shape(T, d, ffn, N * c if N * c < 256 else 256, k, N, c, dtype, act)
        return lz.lz_plan_workspace_bytes(s), lz.lz_ffn_workspace_bytes(s), lz.lz_train_workspace_bytes(s)

    edge = 2 ** 31 // (2 * d)
    tokens = sorted({*range(1, 800), *(int(800 * 1.07 ** i) for i in range(110)), *range(edge - 3, edge + 4)})
    last = (0, 0, 0)
    for T in tokens:
        now = sizes(T)
        # training refuses batches past its limit of row tiles: 0 bytes, no workspace to share
        assert all(n >= l or (n == 0 and i == 2) for i, (n, l) in enumerate(zip(now, last))), (T, now, last)
        last = now


def test_unaligned_forwards_have_a_table_of_the_fp32_kernels_tiles(tmp_path):
    """Sizes that no tile divides take unaligned tensors on the fp32 kernel.  On the padded 256-row table of the bf16
    GEMMs that kernel spends most of its steps on entries without rows (128 slots, 3000 tokens: 4 to 7 times the time),
    so lz_ffn_tiles builds one of 32-row tiles beside it; whole tiles refuse such tensors and need none."""
    out = recorded(tmp_path, """
A, U, out = At(1 << 20), At((1 << 20) + 2), []
for c, T, d, ffn in ((8, 3000, 1000, 2664), (1, 64, 1000, 2664), (8, 3000, 1024, 2560), (8, 3000, 1001, 2664)):
    s = lz.Shape(T, d, ffn, 8, 2, 16, c, lz.LZ_BF16, lz.LZ_SWIGLU)
    n = lz.lz_ffn_workspace_bytes(s)
    rc = [code(lz.lz_expert_ffn, x, A, A, A, s, A, At(1 << 30), n) for x in (A, U)]
    c = [x.split() for x in calls()]
    tables = [int(x[2]) for x in c if "build_tiles" in x[1]]
    gemms = ["f32" if "gemm_f32" in x[1] else "bf16" for x in c if "gemm" in x[1]]
    out.append([rc, tables, gemms])
""")
    assert out[0] == [[0, 0], [2, 2], ["bf16", "bf16", "f32", "bf16"]]    # wide and 32-row tables
    assert out[1] == [[0, 0], [3, 3], ["bf16", "bf16", "f32", "bf16"]]    # and the narrow tiles'
    assert out[2] == [[0, -1], [1, 1], ["bf16", "bf16"]]
    assert out[3] == [[0, 0], [1, 1], ["f32"] * 4]


def test_replica_sums_of_few_short_experts_load_further_ahead(tmp_path):
    """fp32, at most 4 experts in under 1024 workgroups: 16 slots' loads in flight, 4 otherwise."""
    out = recorded(tmp_path, """
A, out = At(1 << 20), []
for S, E, n, dtype in ((512, 1, 65536, lz.LZ_F32), (2048, 4, 1 << 18, lz.LZ_F32), (2048, 4, 255 * 1024, lz.LZ_F32), (512, 5, 65536, lz.LZ_F32),
                       (512, 1, 65536, lz.LZ_BF16), (512, 1, 65534, lz.LZ_F32)):
    rc = code(lz.lz_reduce_replica_grads_dtype, A, A, S, E, n, dtype, A)
    (c,) = calls()
    out.append([rc, "generic" if "generic" in c else c[c.index("kernelI"):][7:12]])
""")
    assert out == [[0, "fLi16"], [0, "fLi4E"], [0, "fLi16"], [0, "fLi4E"], [0, "tLi4E"], [0, "generic"]]


def test_results_of_one_narrow_tile_of_columns_run_on_narrow_tiles(tmp_path):
    """Where all columns fit 64 a 256-wide tile is mostly padding; gated first GEMMs have no narrow form."""
    out = recorded(tmp_path, """
A, out = At(1 << 20), []
for T, d, ffn, act in ((40000, 8, 64, lz.LZ_GELU), (40000, 8, 64, lz.LZ_SWIGLU), (40000, 64, 72, lz.LZ_GELU), (40000, 72, 64, lz.LZ_GELU),
                       (1 << 25, 8, 64, lz.LZ_GELU), ((1 << 25) + 1, 8, 64, lz.LZ_GELU)):
    s = lz.Shape(T, d, ffn, 32, 8 if T > 40000 else 1, 4, 8, lz.LZ_BF16, act)
    rc = code(lz.lz_expert_ffn, A, A, A, A, s, A, At(1 << 30), lz.lz_ffn_workspace_bytes(s))
    out.append([rc] + ["narrow" if "narrow" in c else "wide" for c in calls() if "gemm" in c])
""")
    n, w = "narrow", "wide"
    assert out == [[0, n, n], [0, w, n], [0, w, n], [0, n, w], [0, n, n], [0, w, w]]


def test_the_ragged_wide_tests_run_on_wide_tiles(tmp_path):
    import test_gpu_wide_tiles as wide

    out = recorded(tmp_path, f"""
A, out = At(1 << 20), []
for d, ffn in {wide.SIZES}:
    for act in (lz.LZ_GELU, lz.LZ_SWIGLU):
        s = lz.Shape({sum(wide.COUNTS)}, d, ffn, 64, 1, 1, 64, lz.LZ_BF16, act)
        n = max(lz.lz_ffn_workspace_bytes(s), lz.lz_train_workspace_bytes(s))
        rc = [code(lz.lz_expert_ffn, A, A, A, A, s, A, At(1 << 30), n), code(lz.lz_expert_ffn_gather, A, A, A, A, A, s, A, At(1 << 30), n),
              code(lz.lz_ffn_forward_train, A, A, A, A, s, A, A, A, A, n), code(lz.lz_ffn_backward, A, A, A, A, A, A, A, s, A, A, A, A, n)]
        out.append([rc, sum("gemm_mfma" in c for c in calls())])
        out.append([rc, sum("gemm" in c and "gemm_mfma" not in c for c in calls())])
""")
    assert out[0::2] == [[[0] * 4, 10]] * 4 and out[1::2] == [[[0] * 4, 0]] * 4


def test_the_large_fp32_weight_gradient_tests_run_on_four_waves(tmp_path):
    import test_gpu_f32_sizes as f32

    out = recorded(tmp_path, f"""
A, out = At(1 << 20), []
for d, ffn, slots in {[(d, f, s) for d, f, s in f32.WIDE_GRADIENTS]}:
    s = lz.Shape(1500, d, ffn, 8, 2, 1, slots, lz.LZ_F32, lz.LZ_GELU)
    n = lz.lz_train_workspace_bytes(s)
    rc = [code(f, A, A, A, A, A, A, A, s, A, A, A, A, n) for f in (lz.lz_ffn_backward, lz.lz_ffn_backward_accumulate)]
    names = [c[c.index("kernelIfLi") + 10:] for c in calls() if "gemm_f32" in c]
    out.append([rc, [n[:18] for n in names if n[1:6] == "ELb1E"]])   # WGRAD: both operands k-major
""")
    for (d, ffn, _), (rc, names) in zip(f32.WIDE_GRADIENTS, out):
        vec = "1" if d % 4 == 0 and ffn % 4 == 0 else "0"
        assert rc == [0, 0]
        assert names == [f"{epi}ELb1ELb1ELi4ELb{vec}E" for epi in (0, 0, 5, 5)]


@pytest.mark.parametrize("dtype,d,address", [("LZ_F32", 64, 1 << 20), ("LZ_F32", 1408, 1 << 20), ("LZ_BF16", 65, 1 << 20),
                                             ("LZ_BF16", 64, 1 << 20), ("LZ_BF16", 1408, 1 << 20)])
def test_a_launch_that_fails_ends_the_call(tmp_path, dtype, d, address):
    """Whichever launch of a call fails, the tile tables' among them: the call says so and launches nothing behind it, which
    would read what the failed kernel did not write."""
    out = recorded(tmp_path, f"""
A, W = At({address}), At(1 << 30)
s = lz.Shape(2400, {d}, 1408, 20, 1, 1, 20, lz.{dtype}, lz.LZ_GELU)
n = max(lz.lz_ffn_workspace_bytes(s), lz.lz_train_workspace_bytes(s))
def forward(): return code(lz.lz_expert_ffn, A, A, A, A, s, A, W, n)
def train(): return code(lz.lz_ffn_forward_train, A, A, A, A, s, A, A, A, W, n)
def backward(): return code(lz.lz_ffn_backward, A, A, A, A, A, A, A, s, A, A, A, W, n)
def accumulate(): return code(lz.lz_ffn_backward_accumulate, A, A, A, A, A, A, A, s, A, A, A, W, n)
out = []
for call in (forward, train, backward, accumulate):
    ok, launches = call(), len(calls())
    for i in range(launches):
        fail_launch(i)
        out.append([ok, call(), len(calls()) - i])
""")
    assert len(out) >= 3 + 3 + 5 + 5
    assert out == [[0, -6, 0]] * len(out)    # LZ_EHIP
