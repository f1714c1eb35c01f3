"""ae_step with the exit rule decided on the device, against the rule read back by the host (needs an MI355X)."""
import numpy as np
import pytest

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.binding import AdaEagleError, Engine
from paper_2412_18910_amd.config import BF16, FP32, Config

from .gpu_helpers import to_device

pytestmark = pytest.mark.gpu

# the odd vocabulary of the float32 model leaves exported rows unaligned
CFG = {BF16: Config(2, 256, 4, 2, 64, 512, 1008, dtype=BF16, k_max=5, n_ctx_max=320, ldlp_hidden=64, ddd_enabled=1),
       FP32: Config(2, 264, 4, 2, 64, 712, 1003, dtype=FP32, k_max=5, n_ctx_max=320, ldlp_hidden=64, ddd_enabled=1)}


@pytest.mark.parametrize("dtype", [BF16, FP32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("temperature", [0.0, 0.8])
@pytest.mark.parametrize("theta", [0.5, -0.6, -14.0, -1e9])   # never a token, never past k, now and then, always k_max
def test_step_equals_the_host_rule(dtype, temperature, theta):
    cfg = CFG[dtype].with_(temperature=temperature, ddd_threshold=theta)
    w = to_device(synth.make_weights(cfg, 71))
    ids = synth.token_ids(40, cfg.vocab, 72)
    r = np.random.default_rng(73)
    u = [(r.random(cfg.k_max), r.random(cfg.k_max + 1)) for _ in range(8)]
    runs = []
    for mode in (Engine.DDD_HOST, Engine.DDD_DEVICE):
        eng = Engine(cfg, w)
        eng.set_ddd_mode(mode)
        eng.prefill(ids)
        out = []
        for i, (ud, ua) in enumerate(u):
            k, acc, toks = eng.step(i % (cfg.k_max + 1) if i < 7 else -1, None, ud if temperature else None, ua if temperature else None)
            out.append((k, acc, toks.tolist(), eng.kv_len, [eng.logits(j) for j in range(k + 1)],
                        [eng.draft_logits(j) for j in range(k)]))
        runs.append(out)
        eng.close()
    for a, b in zip(*runs):
        assert a[:4] == b[:4]
        assert all(np.array_equal(x, y) for x, y in zip(a[4] + a[5], b[4] + b[5]))


def test_uniforms_behind_the_drafted_length_are_still_checked():
    cfg = CFG[BF16].with_(temperature=0.8, ddd_threshold=-0.6)
    eng = Engine(cfg, to_device(synth.make_weights(cfg, 71)))
    eng.prefill(synth.token_ids(40, cfg.vocab, 72))
    ua = np.full(cfg.k_max + 1, 0.5)
    ua[-1] = 1.0
    with pytest.raises(AdaEagleError):
        eng.step(1, None, np.full(cfg.k_max, 0.5), ua)
    eng.close()
