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
    out, groups = set(), 0
    for name, gx, *_ in c.launches():
        if m := re.search(r"gemm_f32_dense_kernelILi(\d)ELi(\d)ELb(\d)E", name):
            out.add((EPI[int(m[1])], int(m[2]), int(m[3])))
            groups = gx
        elif m := re.search(r"f32_tail_kernelILi(\d)ELi(\d)E", name):   # the pieces are 512 workgroups at most
            out.add(("TAIL-" + EPI[int(m[1])], int(m[2]), int(groups > 512)))
        elif m := re.search(r"gemm_dense_kernelILi(\d)ELb\dELi(\d)ELi(\d)ELi(\d)E", name):
            out.add((EPI[int(m[1])], int(m[2]), int(m[3]), int(m[4])))
    c.close()
    return out


@pytest.mark.parametrize("name", CASES)
def test_a_case_reaches_the_kernels_it_is_there_for(name):
    assert set(CASES[name].reaches) <= launched(CASES[name])


def test_the_cases_reach_every_kernel():
    f32, bf16 = set(), set()
    for c in CASES.values():
        (bf16 if c.cfg.dtype == BF16 else f32).update(c.reaches)
    tiles = {(e, j, long) for e in ("QKV", "SWIGLU", "PART") for j in (1, 2, 3, 4) for long in (0, 1) if (j, long) != (4, 1)}
    # (64-row tiles alone are split for too few widths to say that it happens)
    tails = {(e, j, whole) for e in ("TAIL-QKV", "TAIL-SWIGLU") for j in (1, 2, 3, 4) for whole in (0, 1) if (j, whole) != (4, 0)}
    assert f32 == tiles | tails
    assert bf16 == {(e, rows, 4, w) for e in ("QKV", "SWIGLU", "RESID", "STORE") for rows, w in ((4, 4), (4, 8), (8, 4))} | \
        {("PART", rows, w, 8) for rows in (4, 8) for w in (2, 3)}


def test_the_widths_end_within_tiles():
    for c in CASES.values():
        if c.cfg.dtype == BF16 and any(r[0] == "QKV" and r[1] != 8 for r in c.reaches):
            assert (c.cfg.n_heads + 2 * c.cfg.n_kv_heads) * c.cfg.head_dim // 16 % 16 == 8
        if any(r[0] in ("RESID", "STORE") and r[-1] == 8 for r in c.reaches):
            assert c.cfg.d_model // 16 % 32 == 16
        assert c.n % 16
