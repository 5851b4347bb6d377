"""Which fp32 GEMMs run on split operands, read from the launches that the library makes, and the barriers of their
kernel, read from its code (no GPU)."""
import re
import subprocess

import pytest

from paper_2407_04656_amd import build

from hip_record import recorded


def test_large_aligned_fp32_forwards_and_weight_gradients_are_split(tmp_path):
    """The sizes of test_gpu_f32_split.py and test_gpu_f32_split_range.py run there; small batches, few rows a slot and
    unaligned tensors do not, and only a forward that reads the table of 64-row tiles builds it (a workgroup per table)."""
    out = recorded(tmp_path, """
A, U, out = At(1 << 20), At((1 << 20) + 4), []
for P, S, d, ffn, w1 in ((2400, 20, 1408, 1408, A), (2400, 20, 1412, 1500, A), (2400, 20, 1412, 1412, A), (2048, 4, 128, 2048, A),
                         (2400, 20, 1408, 1408, U), (256, 20, 1408, 1408, A), (256, 4, 128, 256, A), (2400, 20, 1409, 1408, A),
                         (959, 20, 1408, 1408, A), (960, 20, 1408, 1408, A), (2048, 4, 1024, 1024, A), (2048, 8, 1024, 1024, A)):
    s = lz.Shape(P, d, ffn, S, 1, 1, S, lz.LZ_F32, lz.LZ_GELU)
    n = max(lz.lz_ffn_workspace_bytes(s), lz.lz_train_workspace_bytes(s))
    rc = [code(lz.lz_expert_ffn, A, A, w1, A, s, A, At(1 << 30), n), code(lz.lz_ffn_backward, A, A, A, A, A, w1, A, s, A, A, A, A, n)]
    c = [x.split() for x in calls()]
    out.append([rc, [int(x[2]) for x in c if "build_tiles" in x[1]], "".join("s" if "gemm_split" in x[1] else "f" for x in c if "gemm" in x[1])])
""")
    # up, down, then dZ, dxp, dW2, dW1 of the backward
    assert out == [[[0, 0], [2, 1], "ssffss"], [[0, 0], [2, 1], "ssffss"], [[0, 0], [2, 1], "ssffss"], [[0, 0], [2, 1], "sfffff"],
                   [[0, 0], [2, 1], "fsffss"], [[0, 0], [1, 1], "ffffff"], [[0, 0], [1, 1], "ffffff"], [[0, 0], [2, 1], "ffffff"],
                   [[0, 0], [1, 1], "ffffff"], [[0, 0], [1, 1], "ffffss"], [[0, 0], [1, 1], "ffffff"], [[0, 0], [1, 1], "ffffss"]]


def test_fused_unfused_and_training_forwards_run_on_the_same_kernels(tmp_path):
    """They give the same bits, so where one cannot run on split operands (the fused one reads x through 31-bit offsets) none
    does: the first GEMM's kernel depends on the size of x, not on the call."""
    out = recorded(tmp_path, """
A, W, out = At(1 << 20), At(1 << 30), []
for T in ((1 << 19) - 1, 1 << 19):
    s = lz.Shape(T, 1024, 1024, 8, 1, 1, 8, lz.LZ_F32, lz.LZ_GELU)
    n = max(lz.lz_ffn_workspace_bytes(s), lz.lz_train_workspace_bytes(s))
    for rc in (lambda: code(lz.lz_expert_ffn, A, A, A, A, s, A, W, n), lambda: code(lz.lz_expert_ffn_gather, A, A, A, A, A, s, A, W, n),
               lambda: code(lz.lz_ffn_forward_train, A, A, A, A, s, A, A, A, W, n)):
        out.append([rc(), "".join("s" if "gemm_split" in x else "f" for x in calls() if "gemm" in x)])
""")
    assert out == [[0, "ss"]] * 3 + [[0, "fs"]] * 3


def test_gathered_gated_and_accumulating_calls_are_split_too(tmp_path):
    """The calls of test_gpu_f32_split_range.py, both activations: 2400 rows, 20 slots."""
    out = recorded(tmp_path, """
A, W, out = At(1 << 20), At(1 << 30), []
for act in (lz.LZ_GELU, lz.LZ_SWIGLU):
    s = lz.Shape(2400, 1412, 1500, 20, 1, 1, 20, lz.LZ_F32, act)
    n = max(lz.lz_ffn_workspace_bytes(s), lz.lz_train_workspace_bytes(s))
    rc = [code(lz.lz_expert_ffn_gather, A, A, A, A, A, s, A, W, n), code(lz.lz_ffn_forward_train, A, A, A, A, s, A, A, A, W, n),
          code(lz.lz_ffn_backward_accumulate, A, A, A, A, A, A, A, s, A, A, A, W, n)]
    out.append([rc, "".join("s" if "gemm_split" in x else "f" for x in calls() if "gemm" in x)])
""")
    assert out == [[[0, 0, 0], "ss" + "ss" + "ffss"]] * 2


@pytest.mark.parametrize("epi,wgrad", [("EPI_SWIGLU_KEEP", "false"), ("EPI_ACCUM", "true")])
def test_every_barrier_is_one_for_all_waves(tmp_path, epi, wgrad):
    """A barrier in code that is compiled once for each arm of a branch would be another one for the waves of each arm: the
    kernel's code has as many as its source."""
    text = open(f"{build.CSRC}/gemm_split.h").read()
    kernel = text[text.index("void gemm_split_kernel("):]
    kernel = kernel[:kernel.index("\n}\n")]
    src, asm = tmp_path / "one.hip", tmp_path / "one.s"
    src.write_text(f'#include "gemm_split.h"\nvoid* one() {{ return (void*)gemm_split_kernel<{epi}, {wgrad}>; }}\n')
    done = subprocess.run(["/opt/rocm/bin/hipcc", *build.FLAGS, "-x", "hip", "--cuda-device-only", "-S", str(src), "-o", str(asm)],
                          capture_output=True, text=True)
    assert done.returncode == 0, done.stderr
    code = asm.read_text()
    code = code[re.search(r"^\S*gemm_split_kernel\S*:", code, re.M).end():]
    code = code[:code.index(".Lfunc_end")]
    assert len(re.findall(r"^\s+s_barrier", code, re.M)) == kernel.count("__syncthreads()")
