"""Order of the loads that the float32 GEMMs wait for by count, in the code the compiler makes (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2412_18910_amd import build


@pytest.fixture(scope="module")
def kernels():
    name = "kernels_f32.hip"
    src = os.path.join(build.HERE, "csrc", name)
    asm = subprocess.run(["hipcc", "-S", "--offload-device-only"] + build.COMMON + build.EXTRA[name] + ["-w", "-o", "-", src],
                         check=True, stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, text=True).stdout
    return {m[1]: [line.strip() for line in m[2].splitlines()] for m in re.finditer(r"\n(_ZN2ae\w+):(.*?)\.Lfunc_end", asm, re.S)}


def loads(lines):
    """(into LDS or not, scalar registers of the buffer) of the loads, "wait n", "barrier" and "use" (products) in between"""
    out = []
    for line in lines:
        if line.startswith("buffer_load"):
            out.append(("lds" if line.endswith("lds") else "reg", re.search(r"s\[\d+:\d+\]", line)[0]))
        elif line.startswith("s_waitcnt") and "vmcnt" in line:
            out.append(("wait", int(re.search(r"vmcnt\((\d+)\)", line)[1])))
        elif line.startswith("s_barrier"):
            out.append(("barrier", 0))
        elif line.startswith("v_mfma"):
            out.append(("use", 0))
    return out


def test_decode_gemm_weights_and_activations_take_turns(kernels):
    names = [n for n in kernels if "15gemm_f32_kernel" in n]
    assert names
    for n in names:
        kinds = [k for k, _ in loads(kernels[n]) if k in ("lds", "reg")]
        w = 4 if "kernelILi2E" in n else 2   # gate/up: two matrices
        half = ["lds"] * w + ["reg"] * 2
        assert kinds[:4 * len(half)] == half * 4, n   # both halves of the first chunk, and of the loop


def test_prompt_gemm_weights_are_the_newest_loads_at_every_barrier(kernels):
    names = [n for n in kernels if "21gemm_f32_dense_kernel" in n]
    assert names
    for n in names:
        seq = loads(kernels[n])
        seq = seq[:max(i for i, x in enumerate(seq) if x[0] == "barrier")]
        stage, stages, first = [], 0, None
        for kind, what in seq:
            if kind == "lds":
                stage.append(what)
            elif kind == "barrier":
                weights = set(stage[-4:])
                first = first or weights
                assert weights == first and len(weights) == 2, n      # the two matrix blocks, two loads each
                assert all(s not in weights for s in (stage[:-4] if stages else stage[8:-4])), n
                stage, stages = [], stages + 1
        assert stages >= 6, n
