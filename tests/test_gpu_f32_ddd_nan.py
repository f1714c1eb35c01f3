"""Float32 exit rule with a logit that is not a number (needs an MI355X)."""
import numpy as np
import pytest

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.binding import Engine
from paper_2412_18910_amd.config import FP32, Config

from .gpu_helpers import to_device

pytestmark = pytest.mark.gpu

CFG = Config(2, 264, 4, 2, 64, 712, 1003, dtype=FP32, k_max=5, n_ctx_max=128, ldlp_hidden=64, ddd_enabled=1, ddd_threshold=-1e9)


@pytest.mark.parametrize("value", [float("nan"), float("inf"), None])
@pytest.mark.parametrize("token", [0, 500, 1002])   # row-blocks at either end, the ragged last one
def test_a_statistic_that_is_no_number_ends_the_draft(value, token):
    """log p is NaN with such a logit in the softmax, NaN >= theta is false: nothing is drafted past k.  (None: the
    rule goes on to k_max.)"""
    w = synth.make_weights(CFG, 97)
    if value is not None:
        w["lm_head"][token] = value   # an Inf row: logits of Inf or NaN by the signs of the features
    eng = Engine(CFG, to_device(w))
    ids = synth.token_ids(30, CFG.vocab, 98)
    ids[ids == token] = 3
    for mode in (Engine.DDD_HOST, Engine.DDD_DEVICE):
        eng.prefill(ids)
        eng.set_ddd_mode(mode)
        d = eng.draft(2, override_ids=np.full(CFG.k_max, 4, np.int32))
        assert len(d) == (CFG.k_max if value is None else 2)
        assert np.isnan(eng.draft_logprob) == (value is not None)
    eng.close()
