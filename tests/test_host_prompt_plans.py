"""Which prompt GEMMs the cases of test_gpu_prompt_plans.py launch, and the rows of a chunk (host code over a recorded HIP runtime,
no GPU)."""
import pytest

from paper_2412_18910_amd.binding import AE_ENOMEM, AE_OK
from paper_2412_18910_amd.config import BF16, FP32, Config

from .fake_runtime import Ctx
from .test_gpu_prompt_plans import CASES, _cfg
from .test_gpu_prompt_tiles import Case
from .test_host_prompt_tiles import launched


def test_the_cases_reach_the_kernels_they_are_there_for():
    # (all of them together: constants fitted anew may change which case it is)
    out = set().union(*(launched(Case(_cfg(*widths), n, (), chunk=8192)) for widths, n, _ in CASES))
    assert set().union(*(reaches for *_, reaches in CASES)) <= out


@pytest.mark.parametrize("d,heads,kv,ffn", [(256, 2, 1, 256), (256, 4, 4, 4096), (512, 4, 2, 11008), (768, 8, 8, 4096), (1024, 16, 8, 2816),
                                            (3072, 16, 16, 6144), (3072, 48, 16, 4096), (4096, 4, 2, 4096), (4096, 32, 32, 11008),
                                            (4096, 32, 8, 14336), (4352, 8, 8, 4352), (5120, 40, 40, 13824)])
def test_every_plan_is_launched(d, heads, kv, ffn):
    cfg = Config(1, d, heads, kv, 128, ffn, 512, dtype=BF16, k_max=5, n_ctx_max=8300, ldlp_hidden=64)
    c = Ctx(cfg)
    assert c.prefill_mode(0, 8192) == AE_OK
    for n in sorted({int(17 * 1.07 ** i) for i in range(91)} | {64, 128, 2048, 4096, 8192}, reverse=True):
        c.lib.fake_clear()
        assert c.prefill(n) == AE_OK
        names = [x[0] for x in c.launches()]
        # QKV, o, gate/up and down of the layer, the draft head's input and QKV projections
        assert sum("gemm_dense_kernel" in x for x in names) == 6, n
        whole = sum("gemm_dense_kernel" in x and "gemm_dense_kernelILi4E" not in x for x in names)
        assert whole + sum("dense_sum_rows_kernel" in x or "dense_finish_kernel" in x for x in names) == 6, n
    c.close()


def chunks(cfg, n, chunk=0, limit=0):
    c = Ctx(cfg)
    assert c.prefill_mode(0, chunk) == AE_OK
    c.lib.fake_fail_alloc(limit)
    c.lib.fake_clear()
    rc = c.prefill(n)
    out = sum("embed_dense_kernel" in name or "embed_f32_kernel" in name for name, *_ in c.launches())
    c.lib.fake_fail_alloc(0)
    c.close()
    return rc, out


def test_rows_of_a_chunk():
    cfg = Config(1, 512, 8, 2, 64, 1024, 512, dtype=BF16, k_max=4, n_ctx_max=8300, ldlp_hidden=64)
    assert chunks(cfg, 2049) == chunks(cfg, 4096) == (AE_OK, 1)
    assert chunks(cfg, 4097) == (AE_OK, 2) and chunks(cfg, 8200) == (AE_OK, 3)
    assert chunks(cfg, 8200, chunk=2048) == (AE_OK, 5)
    assert chunks(cfg.with_(dtype=FP32), 4096) == (AE_OK, 2)
    # no room for 4096 rows: the 2048 that there is room for, unless the caller has asked for more
    room = 2048 * cfg.d_ffn * 4 + 1
    assert chunks(cfg, 8200, limit=room) == (AE_OK, 5)
    assert chunks(cfg, 8200, chunk=4096, limit=room)[0] == AE_ENOMEM
    assert chunks(cfg, 8200, limit=room - 1)[0] == AE_ENOMEM
