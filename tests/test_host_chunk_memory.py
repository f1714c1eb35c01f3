"""Chunks of a prompt where memory is short: what did not fit is not asked for again, and buffers that do are not given up (host code
over a recorded HIP runtime, no GPU)."""
import pytest

from paper_2412_18910_amd.binding import AE_ENOMEM, AE_OK
from paper_2412_18910_amd.config import BF16, FP32, Config

from .fake_runtime import Ctx

CFG = Config(1, 512, 8, 2, 64, 1024, 512, dtype=BF16, k_max=4, n_ctx_max=8300, ldlp_hidden=64)


@pytest.fixture
def make():
    made = []

    def f(cfg=CFG):
        made.append(Ctx(cfg))
        return made[-1]
    yield f
    for c in made:
        c.lib.fake_fail_alloc(0)
        c.lib.fake_room(0)
        c.close()


def run(c, n):
    """(result, chunks, buffers cleared) of a prompt."""
    c.lib.fake_clear()
    rc = c.prefill(n)
    names = [x[0] for x in c.launches()]
    assert c.lib.fake_last_error() == 0
    return rc, sum("embed_dense_kernel" in x or "embed_f32_kernel" in x for x in names), sum("fill_zero" in x for x in names)


def test_a_chunk_that_did_not_fit_is_not_tried_again(make):
    c = make()
    c.lib.fake_fail_alloc(2048 * CFG.d_ffn * 4 + 1)   # the FFN rows of 2048, not of 4096
    rc, chunks, cleared = run(c, 8200)
    assert (rc, chunks) == (AE_OK, 5) and cleared > 0
    held = c.lib.fake_live_bytes()
    assert run(c, 8200) == (AE_OK, 5, 0) and run(c, 2100) == (AE_OK, 2, 0)
    assert c.lib.fake_live_bytes() == held


def test_memory_that_is_free_again_is_used_when_the_mode_is_set(make):
    c = make()
    c.lib.fake_fail_alloc(2048 * CFG.d_ffn * 4 + 1)
    assert run(c, 8200)[:2] == (AE_OK, 5)
    c.lib.fake_fail_alloc(0)
    assert run(c, 8200) == (AE_OK, 5, 0)   # as before: a prompt's sums do not depend on what is free
    assert c.prefill_mode(0) == AE_OK
    assert run(c, 8200)[:2] == (AE_OK, 3)


def test_buffers_that_will_do_are_kept_until_larger_ones_are_there(make):
    c = make()
    assert run(c, 2048)[:2] == (AE_OK, 1)
    held = c.lib.fake_live_bytes()
    c.lib.fake_room(held + 4096)   # memory has become tight
    for n, chunks in ((3000, 2), (8200, 5), (2048, 1), (100, 1)):
        assert run(c, n) == (AE_OK, chunks, 0)
        assert c.lib.fake_live_bytes() == held


def test_a_context_between_both_sizes_keeps_what_it_has(make):
    c = make()
    assert run(c, 2500)[:2] == (AE_OK, 1)
    c.lib.fake_room(c.lib.fake_live_bytes() + 4096)
    assert run(c, 8200) == (AE_OK, 4, 0) and run(c, 8200) == (AE_OK, 4, 0)   # 2560 rows each


def test_larger_buffers_take_the_place_of_smaller_ones(make):
    c, fresh = make(), make()
    base = c.lib.fake_live_bytes()
    assert run(fresh, 8200)[:2] == (AE_OK, 3)
    whole = c.lib.fake_live_bytes() - base
    assert run(c, 2048)[:2] == (AE_OK, 1) and run(c, 8200)[:2] == (AE_OK, 3)
    assert c.lib.fake_live_bytes() - base == 2 * whole


def test_pieces_of_k_weigh_more_than_the_larger_chunk(make):
    # room for 4096 rows without the pieces, or for 2048 with them
    c = make()
    base = c.lib.fake_live_bytes()
    assert run(c, 4096)[:2] == (AE_OK, 1)
    c.lib.fake_room(c.lib.fake_live_bytes() - 1)
    c.close()
    c.__init__(CFG)
    assert c.lib.fake_live_bytes() == base
    assert run(c, 4096)[:2] == (AE_OK, 2)
    c.lib.fake_clear()
    assert c.prefill(100) == AE_OK
    assert any("dense_sum_rows_kernel" in x[0] for x in c.launches())


def test_a_chunk_that_the_caller_set_is_taken_as_set(make):
    c = make()
    assert c.prefill_mode(0, 4096) == AE_OK
    c.lib.fake_fail_alloc(2048 * CFG.d_ffn * 4 + 1)
    for _ in range(2):
        assert run(c, 8200)[0] == AE_ENOMEM
    assert c.prefill_mode(0, 2048) == AE_OK
    assert run(c, 8200)[:2] == (AE_OK, 5)


def test_float32_chunks_of_two_thirds_stay(make):
    cfg = CFG.with_(dtype=FP32, n_ctx_max=2400)
    c = make(cfg)
    c.lib.fake_fail_alloc(2048 * cfg.d_ffn * 4 + 1)   # a float an activation, not three parts
    assert run(c, 2048)[:2] == (AE_OK, 2)
    held = c.lib.fake_live_bytes()
    c.lib.fake_room(held)
    c.lib.fake_fail_alloc(1)   # nothing more can be had
    assert run(c, 2048)[:2] == (AE_OK, 2) and run(c, 1100)[:2] == (AE_OK, 1)
    assert c.lib.fake_live_bytes() == held
