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


# widths whose last tiles are made in pieces of K, which go where a short prompt's buffer has little room
@pytest.mark.parametrize("heads,kv,hd,d,ffn", [(32, 8, 64, 2048, 5632), (32, 8, 64, 2048, 8192), (16, 8, 64, 1024, 2816),
                                               (16, 8, 64, 1024, 4096), (16, 8, 64, 1032, 4104)])
def test_short_float32_prompts_run_alike_in_fresh_and_used_contexts(heads, kv, hd, d, ffn):
    cfg = Config(1, d, heads, kv, hd, ffn, 512, dtype=FP32, k_max=5, n_ctx_max=2100, ldlp_hidden=64)
    used = {}
    for before in (300, 1500, 2048):
        used[before] = Ctx(cfg)
        assert used[before].prefill(before) == AE_OK
    for n in range(17, 260, 3):
        out = {}
        for before, c in [(0, Ctx(cfg)), *used.items()]:
            c.lib.fake_clear()
            assert c.prefill(n) == AE_OK
            out[before] = [x for x in c.launches() if "fill_zero" not in x[0]]
            if not before:
                c.close()
        assert all(x == out[0] for x in out.values()), n
    for c in used.values():
        c.close()
