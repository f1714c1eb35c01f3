"""How long a call polls for the device before it sleeps on the stream (host code over a recorded HIP runtime, no GPU)."""
import time

import pytest

from paper_2412_18910_amd.binding import AE_EHIP, AE_OK
from paper_2412_18910_amd.config import TINY

from .fake_runtime import Ctx


@pytest.fixture
def ctx():
    c = Ctx(TINY)
    assert c.prefill(20) == AE_OK
    yield c
    c.lib.fake_mute(0)
    c.close()


def test_a_wait_without_an_answer_sleeps_after_10_ms(ctx):
    """The core is burnt for 10 ms at most (CPU time of the thread, whatever else the machine does)."""
    ctx.lib.fake_mute(1)
    assert ctx.verify(1) == AE_OK
    before, t = ctx.lib.fake_syncs(), time.thread_time()
    assert ctx.accept() == AE_EHIP
    assert ctx.lib.fake_syncs() == before + 1
    assert time.thread_time() - t < 0.025
