"""Rows on their way to the host: which fetches launch what (host code over a recorded HIP runtime, no GPU), and the memory
they are returned in."""
import pytest

from paper_2412_18910_amd.binding import AE_EHIP, AE_OK, AdaEagleError, Engine
from paper_2412_18910_amd.config import BF16, FP32, Config

from .fake_runtime import Ctx


@pytest.fixture(params=[BF16, FP32], ids=["bf16", "fp32"])
def ctx(request):
    cfg = Config(1, 256, 4, 2, 64, 512, 515 if request.param == FP32 else 512, dtype=request.param, k_max=5, n_ctx_max=128, ldlp_hidden=64)
    c = Ctx(cfg)
    assert c.prefill(20) == AE_OK
    yield c
    c.close()


def test_only_a_second_row_in_order_brings_the_next_one(ctx):
    n = ctx.count
    assert n(lambda: ctx.verify(4)) > 0
    assert [n(lambda: ctx.logits(i)) for i in (0, 1, 2, 3)] == [1, 2, 1, 0]
    assert [n(lambda: ctx.logits(i)) for i in (0, 0, 2, 3, 1)] == [1, 1, 1, 1, 1]   # 3 follows 2, but is the last
    assert [n(lambda: ctx.logits(i)) for i in (0, 1, 3, 2)] == [1, 2, 1, 1]          # 2 came for nothing
    assert [n(lambda: ctx.logits(i)) for i in (3, 4, 5)] == [1, 1, 1]                # behind the block


def test_a_row_ahead_is_dropped_by_whatever_writes_rows(ctx):
    n = ctx.count
    for again in (lambda: ctx.verify(4), lambda: ctx.draft(3) or ctx.verify(4), lambda: ctx.prefill(20) or ctx.verify(4)):
        assert ctx.verify(4) == AE_OK
        assert [n(lambda: ctx.logits(i)) for i in (0, 1)] == [1, 2]
        assert again() == AE_OK
        assert [n(lambda: ctx.logits(i)) for i in (2, 3)] == [1, 1]
    for other in (lambda: ctx.feature(0), ctx.kv_row):
        assert [n(lambda: ctx.logits(i)) for i in (0, 1)] == [1, 2]
        assert other() == AE_OK
        assert n(lambda: ctx.logits(2)) == 1


@pytest.mark.parametrize("before", [0, 1, 2])   # rows fetched in order before the capture: none sent ahead, one that would be, one that is
def test_a_fetch_under_capture_is_refused_and_leaves_nothing_behind(ctx, before):
    assert ctx.verify(5) == AE_OK
    assert [ctx.logits(i) for i in range(before)] == [AE_OK] * before
    ctx.lib.fake_capture(1)
    assert ctx.logits(before) == AE_EHIP
    ctx.lib.fake_capture(0)
    ctx.lib.fake_set_error(0)   # of the wait that was refused
    assert [ctx.logits(i) for i in (before + 1, before + 2, before, 0)] == [AE_OK] * 4


def test_a_row_that_could_not_be_sent_ahead_is_sent_when_it_is_fetched(ctx):
    n = ctx.count
    assert ctx.verify(4) == AE_OK and ctx.logits(0) == AE_OK
    ctx.lib.fake_fail_launch(1)
    assert ctx.logits(1) == AE_OK and ctx.lib.fake_last_error() == 0
    assert [n(lambda: ctx.logits(i)) for i in (2, 3)] == [2, 0] and ctx.accept() == AE_OK


def test_rows_are_the_callers_own(ctx):
    eng = Engine.__new__(Engine)   # (an engine's weights are on a GPU)
    eng.lib, eng.cfg, eng.h = ctx.lib, ctx.cfg, ctx.h
    try:
        assert ctx.verify(4) == AE_OK
        rows = [eng.logits(i % 4) for i in range(100)] + [eng.feature(0), eng.kv_row(0, 0, 0)]
        assert all(r.flags.owndata and r.flags.writeable for r in rows) and len({r.ctypes.data for r in rows}) == len(rows)
        rows[0].resize(2 * len(rows[0]), refcheck=False)
        with pytest.raises(AdaEagleError):
            eng.logits(99)
    finally:
        eng.h = None
