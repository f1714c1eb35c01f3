"""A prompt runs the same kernels whatever prompts came before it (host code over a recorded HIP runtime, no GPU)."""
import pytest

from paper_2412_18910_amd.binding import AE_OK
from paper_2412_18910_amd.config import BF16, FP32, Config

from .fake_runtime import Ctx


@pytest.mark.parametrize("dtype", [BF16, FP32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("chunk", [128, 2048, 8192])
def test_launches_do_not_depend_on_earlier_prompts(dtype, chunk):
    cfg = Config(1, 2048, 8, 4, 128, 2816, 512, dtype=dtype, k_max=5, n_ctx_max=8300, ldlp_hidden=64)
    lengths = (20, 100, 200, 333, 700, 1100, 2048)

    def run(before):
        c = Ctx(cfg)
        assert c.prefill_mode(0, chunk) == AE_OK
        out = []
        for n in lengths:
            assert before is None or c.prefill(before) == AE_OK
            c.lib.fake_clear()
            assert c.prefill(n) == AE_OK
            out.append([x for x in c.launches() if "fill_zero" not in x[0]])
        c.close()
        return out

    fresh = []
    for n in lengths:   # a context of its own each
        c = Ctx(cfg)
        assert c.prefill_mode(0, chunk) == AE_OK
        c.lib.fake_clear()
        assert c.prefill(n) == AE_OK
        fresh.append([x for x in c.launches() if "fill_zero" not in x[0]])
        c.close()
    for before in (None, 300, 5000, 8000):
        for n, a, b in zip(lengths, fresh, run(before)):
            assert a == b, (before, n)
