"""Prompt buffers that cannot be allocated (host code over a recorded HIP runtime, no GPU)."""
import pytest

from paper_2412_18910_amd.binding import AE_ENOMEM, AE_OK
from paper_2412_18910_amd.config import BF16, Config, TINY

from .fake_runtime import Ctx

MID = Config(2, 512, 8, 2, 64, 1024, 1024, dtype=BF16, k_max=4, n_ctx_max=2400, ldlp_hidden=64)


@pytest.fixture
def make():
    made = []

    def f(cfg):
        made.append(Ctx(cfg))
        return made[-1]
    yield f
    for c in made:
        c.lib.fake_fail_alloc(0)
        c.close()


def names(c):
    return "\n".join(n for n, *_ in c.launches())


@pytest.mark.parametrize("n", [20, 100, 300, 2048])
def test_no_room_for_pieces_of_k_is_no_reason_to_refuse_a_prompt(make, n):
    c = make(MID)
    c.lib.fake_clear()
    assert c.prefill(n) == AE_OK
    split = "dense_sum_rows_kernel" in names(c)
    c.close()
    c.__init__(MID)
    # the pieces are the largest buffer: 16 times the widest output or 768 tiles of 128 x 128
    cap = (n + 127) // 128 * 128
    c.lib.fake_fail_alloc(min(16 * cap * 2 * MID.d_ffn, 768 * 128 * 128) * 4)
    c.lib.fake_clear()
    assert c.prefill(n) == AE_OK
    k = names(c)
    assert "gemm_dense_kernel" in k and "attn_prefill_kernel" in k and split
    assert "dense_sum_rows_kernel" not in k and "dense_finish_kernel" not in k and "gemm_dense_kernelILi4E" not in k
    assert c.lib.fake_last_error() == 0


def test_a_refused_prompt_holds_no_memory(make):
    c = make(MID)
    base = c.lib.fake_live_bytes()
    c.lib.fake_fail_alloc(2048 * 1024 * 4)   # the FFN rows: the buffers before them are there already
    assert c.prefill(2048) == AE_ENOMEM
    assert c.lib.fake_live_bytes() == base and c.lib.fake_last_error() == 0
    c.lib.fake_fail_alloc(0)
    assert c.prefill(2048) == AE_OK and c.lib.fake_live_bytes() > base


@pytest.mark.parametrize("limit", [1, 300 * 256 * 4, 300 * 688 * 4, 2048 * 256 * 4])   # from the first buffer to the last
def test_float32_goes_back_to_blocks_and_holds_no_memory(make, limit):
    c = make(TINY)
    base = c.lib.fake_live_bytes()
    c.lib.fake_fail_alloc(limit)
    for _ in range(2):
        c.lib.fake_clear()
        assert c.prefill(300) == AE_OK
        k = names(c)
        assert "attn_f32_kernel" in k and "attn_prefill_f32_kernel" not in k
        assert c.lib.fake_live_bytes() == base and c.lib.fake_last_error() == 0
    c.lib.fake_fail_alloc(0)
    c.lib.fake_clear()
    assert c.prefill(300) == AE_OK and "attn_prefill_f32_kernel" in names(c)


@pytest.mark.parametrize("n", [700, 1100, 2048])
def test_float32_planes_that_do_not_fit_take_smaller_chunks(make, n):
    cfg = TINY.with_(n_ctx_max=2400)
    c = make(cfg)
    # room for a float an activation (K in whole k-tiles of 32), not for three parts
    c.lib.fake_fail_alloc((n + 127) // 128 * 128 * ((cfg.d_ffn + 31) // 32 * 32) * 4 + 1)
    for _ in range(2):
        c.lib.fake_clear()
        assert c.prefill(n) == AE_OK and c.lib.fake_last_error() == 0
        k = names(c)
        assert "attn_prefill_f32_kernel" in k and "attn_f32_kernel" not in k
        assert k.count("embed_f32_kernel") == 2


def test_a_failed_larger_prompt_leaves_the_shorter_ones_working(make):
    for cfg in (MID, TINY.with_(n_ctx_max=2400)):
        c = make(cfg)
        assert c.prefill(100) == AE_OK
        c.lib.fake_fail_alloc(1024 * cfg.d_model * 4)
        assert c.prefill(2000) == (AE_ENOMEM if cfg.dtype == BF16 else AE_OK)
        assert c.prefill(100) == AE_OK
        c.lib.fake_fail_alloc(0)


@pytest.mark.parametrize("cfg", [MID, TINY], ids=["bf16", "fp32"])
def test_prompt_buffers_are_on_the_device_of_the_context(make, cfg):
    c = make(cfg)
    c.lib.fake_set_device(1)   # the thread has moved on to another GPU
    assert c.prefill(100) == AE_OK
    assert c.lib.fake_malloc_device() == 0 and c.lib.fake_device() == 1
    c.lib.fake_set_device(0)
