"""ae_step with the exit rule on the device, at widths whose next projection is enqueued ahead of the decision (needs an
MI355X)."""
import numpy as np
import pytest

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.binding import Engine
from paper_2412_18910_amd.config import BF16, FP32, Config

from .gpu_helpers import to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [BF16, FP32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("theta", [-0.6, -14.0, -1e9])   # never past k, now and then, always k_max
def test_step_equals_the_host_rule(dtype, theta):
    cfg = Config(1, 2048, 4, 2, 64, 512, 1008, dtype=dtype, k_max=5, n_ctx_max=320, ldlp_hidden=64, ddd_enabled=1, ddd_threshold=theta)
    w = to_device(synth.make_weights(cfg, 75))
    ids = synth.token_ids(40, cfg.vocab, 76)
    runs = []
    for mode in (Engine.DDD_HOST, Engine.DDD_DEVICE):
        eng = Engine(cfg, w)
        eng.set_ddd_mode(mode)
        eng.prefill(ids)
        out = []
        for i in range(8):
            k, acc, toks = eng.step(i % (cfg.k_max + 1))
            out.append((k, acc, toks.tolist(), eng.kv_len, [eng.logits(j) for j in range(k + 1)], [eng.draft_logits(j) for j in range(k)]))
        runs.append(out)
        eng.close()
    for a, b in zip(*runs):
        assert a[:4] == b[:4]
        assert all(np.array_equal(x, y) for x, y in zip(a[4] + a[5], b[4] + b[5]))
