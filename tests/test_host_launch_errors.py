"""A launch that fails is reported, by the call that made it or (an error that was pending before) by the next
acceptance; no call drops one.  Host code over a recorded HIP runtime, no GPU."""
import pytest

from paper_2412_18910_amd.binding import AE_EHIP, AE_OK
from paper_2412_18910_amd.config import BF16, Config, TINY

from .fake_runtime import Ctx

SMALL = Config(2, 256, 4, 2, 64, 512, 1024, dtype=BF16, k_max=4, n_ctx_max=320, ldlp_hidden=64)
FOREIGN = 1   # hipErrorInvalidValue of some other call of the application


@pytest.fixture(params=[SMALL, TINY], ids=["bf16", "fp32"])
def ctx(request):
    c = Ctx(request.param)
    assert c.prefill(20) == AE_OK
    yield c
    c.lib.fake_fail_launch(-1)
    c.lib.fake_set_error(0)
    c.close()


def test_every_failed_launch_of_a_verification_is_reported(ctx):
    n = ctx.count(lambda: ctx.verify(3))
    for i in range(n):
        ctx.lib.fake_fail_launch(i)
        results = [ctx.verify(3), ctx.logits(0), ctx.accept()]
        assert results[0] == AE_EHIP and results[2] != AE_OK, (i, results)
        assert ctx.verify(3) == AE_OK and ctx.logits(0) == AE_OK and ctx.accept() == AE_OK
        assert ctx.set_state(20) == AE_OK


def test_every_failed_launch_of_a_draft_is_reported(ctx):
    assert ctx.set_state(20) == AE_OK
    n = ctx.count(lambda: ctx.draft(3))
    for i in range(n):
        assert ctx.set_state(20) == AE_OK
        ctx.lib.fake_fail_launch(i)
        assert ctx.draft(3) == AE_EHIP, i
        assert ctx.logits(0) == AE_OK
        # nothing of the failed draft is left: it can be made again
        assert ctx.draft(3) == AE_OK and ctx.verify(4, implicit=True) == AE_OK and ctx.accept() == AE_OK


@pytest.mark.parametrize("call", ["logits", "feature", "kv_row", "set_state"])
def test_an_error_that_was_pending_stays_for_the_acceptance(ctx, call):
    between = (lambda: ctx.set_state(20)) if call == "set_state" else getattr(ctx, call)
    assert ctx.set_state(20) == AE_OK and ctx.draft(2) == AE_OK and ctx.verify(3, implicit=True) == AE_OK
    ctx.lib.fake_set_error(FOREIGN)
    assert between() == AE_OK
    assert ctx.lib.fake_last_error() == FOREIGN
    if call == "set_state":
        assert ctx.draft(2) == AE_OK and ctx.verify(3, implicit=True) == AE_OK
    assert ctx.accept() == AE_EHIP


@pytest.mark.parametrize("call", ["logits", "feature", "kv_row", "set_state"])
@pytest.mark.parametrize("pending", [0, FOREIGN])
def test_a_getter_reports_its_own_launches(ctx, call, pending):
    fn = (lambda: ctx.set_state(30)) if call == "set_state" else getattr(ctx, call)
    n = ctx.count(fn)
    for i in range(n):
        assert ctx.set_state(20) == AE_OK
        ctx.lib.fake_set_error(pending)
        ctx.lib.fake_fail_launch(i)
        assert fn() == AE_EHIP, i
        assert ctx.lib.ae_kv_len(ctx.h) == 20
        assert ctx.lib.fake_last_error() == 0   # reported once
        assert fn() == AE_OK
