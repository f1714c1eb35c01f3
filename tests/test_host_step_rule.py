"""What ae_step enqueues around the exit rule's decisions (host code over a recorded HIP runtime, no GPU)."""
import pytest

from paper_2412_18910_amd.binding import AE_OK
from paper_2412_18910_amd.config import BF16, FP32, Config

from .fake_runtime import Ctx


@pytest.mark.parametrize("dtype", [BF16, FP32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("go_on", [0, 1])
@pytest.mark.parametrize("k", [0, 1, 3, 5])
def test_the_next_projection_of_a_wide_model_goes_ahead_of_the_decision(dtype, go_on, k):
    """A rule that stops behind the first decision costs one launch that returns at once, one that goes on none."""
    counts = {}
    for d in (256, 2048):
        c = Ctx(Config(1, d, 4, 2, 64, 512, 1024, dtype=dtype, k_max=5, n_ctx_max=320, ldlp_hidden=64, ddd_enabled=1, ddd_threshold=-1.0))
        assert c.prefill(20) == AE_OK
        c.lib.fake_rule(go_on)
        c.lib.fake_clear()
        rc, io = c.step(k)
        assert rc == AE_OK and io.k == (5 if go_on else max(k, 1))
        counts[d] = c.lib.fake_launches()
        c.lib.fake_rule(1)
        c.close()
    assert counts[2048] - counts[256] == (1 if not go_on and k < 5 else 0)
