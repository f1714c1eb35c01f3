"""Which prompt GEMMs the cases of test_gpu_prompt_tiles.py launch (host code over a recorded HIP runtime, no GPU)."""
import re

import pytest

from paper_2412_18910_amd.binding import AE_OK
from paper_2412_18910_amd.config import BF16

from .fake_runtime import Ctx
from .test_gpu_prompt_tiles import CASES

EPI = {0: "STORE", 1: "RESID", 2: "SWIGLU", 3: "QKV", 4: "PART"}


def launched(case):
    c = Ctx(case.config)
    assert c.prefill_mode(0, case.chunk) == AE_OK
    c.lib.fake_clear()
    assert c.prefill(case.n) == AE_OK
    out = set()
    for name, *_ in c.launches():
        m = re.search(r"gemm_f32_dense_kernelILi(\d)ELi(\d)ELb(\d)E", name) or \
            re.search(r"gemm_dense_kernelILi(\d)ELb\dELi(\d)ELi(\d)ELi\dE", name)
        if m:
            out.add((EPI[int(m[1])], int(m[2]), int(m[3])))
    c.close()
    return out


@pytest.mark.parametrize("name", CASES)
def test_a_case_reaches_the_kernels_it_is_there_for(name):
    assert set(CASES[name].reaches) <= launched(CASES[name])


def test_the_cases_reach_every_kernel():
    f32, bf16 = set(), set()
    for c in CASES.values():
        (bf16 if c.cfg.dtype == BF16 else f32).update(c.reaches)
    assert f32 == {(e, j, long) for e in ("QKV", "SWIGLU", "PART") for j in (1, 2, 3, 4) for long in (0, 1) if (j, long) != (4, 1)}
    assert bf16 == {(e, rows, 4) for e in ("QKV", "SWIGLU", "RESID", "STORE") for rows in (4, 8)} | \
        {("PART", rows, w) for rows in (4, 8) for w in (2, 3)}
