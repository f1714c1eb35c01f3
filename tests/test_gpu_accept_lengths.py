"""Greedy acceptance of every length, beside the LDLP's input layer and as a kernel of its own (needs an MI355X)."""
import numpy as np
import pytest

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.binding import Engine
from paper_2412_18910_amd.config import BF16, FP32, Config

from .gpu_helpers import to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [BF16, FP32], ids=["bf16", "fp32"])
def test_every_prefix_is_accepted(dtype):
    cfg = Config(2, 256, 4, 2, 64, 512, 1008, dtype=dtype, k_max=15, n_ctx_max=128, ldlp_hidden=64)
    eng = Engine(cfg, to_device(synth.make_weights(cfg, 81)))
    ids = synth.token_ids(30, cfg.vocab, 82)
    eng.prefill(ids)
    chain = [eng.pending]   # the target's own continuation, a token a pass
    for _ in range(16):
        eng.verify([chain[-1]])
        assert eng.accept()[0] == 0   # no draft: the acceptance has a launch of its own
        chain.append(eng.pending)
    for a in range(16):
        draft = np.array(chain[1:16], np.int32)
        if a < 15:
            draft[a] = (draft[a] + 1) % cfg.vocab
        eng.prefill(ids)
        assert eng.pending == chain[0]
        k, acc, toks = eng.step(15, draft)
        assert (k, acc, toks.tolist()) == (15, a, chain[1:a + 2]) and eng.kv_len == 31 + a
        k_next = eng.ldlp()
        eng.prefill(ids)
        eng.verify(np.concatenate([[chain[0]], draft]).astype(np.int32))
        assert eng.accept() == (a, chain[a + 1]) and eng.kv_len == 31 + a
        assert eng.ldlp() == k_next   # from the history and features that the acceptance left
    eng.close()
