"""Which prompt GEMMs the cases of test_gpu_prompt_plans.py launch, and the rows of a chunk (host code over a recorded HIP runtime,
no GPU)."""
import pytest

from paper_2412_18910_amd.binding import AE_ENOMEM, AE_OK
from paper_2412_18910_amd.config import BF16, FP32, Config

from .fake_runtime import Ctx
from .test_gpu_prompt_plans import CASES, _cfg
from .test_gpu_prompt_tiles import Case
from .test_host_prompt_tiles import launched


@pytest.mark.parametrize("widths,n,reaches", CASES)
def test_a_case_reaches_the_kernels_it_is_there_for(widths, n, reaches):
    assert reaches <= launched(Case(_cfg(*widths), n, (), chunk=8192))


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
