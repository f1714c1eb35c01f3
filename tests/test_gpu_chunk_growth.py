"""Chunk buffers that take the place of smaller ones while these are still held (needs an MI355X)."""
import numpy as np
import pytest

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.binding import Engine
from paper_2412_18910_amd.config import BF16, Config

from .gpu_helpers import to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths", [(2048, 4097), (100, 2048, 3001), (2500, 4096, 8200)])
def test_a_prompt_gives_the_same_bits_in_a_used_context(lengths):
    cfg = Config(1, 512, 8, 2, 64, 1024, 512, dtype=BF16, k_max=4, n_ctx_max=8300, ldlp_hidden=64)
    w = to_device(synth.make_weights(cfg, 121))
    used = Engine(cfg, w)
    for n in lengths:
        ids = synth.token_ids(n, cfg.vocab, n)
        fresh = Engine(cfg, w)
        for eng in (used, fresh):
            eng.prefill(ids)
        assert np.array_equal(used.logits(0), fresh.logits(0)) and used.pending == fresh.pending
        for layer in (0, 1):
            for slot in {0, n // 2, n - 2}:
                assert np.array_equal(used.kv_row(layer, 1, slot), fresh.kv_row(layer, 1, slot))
        fresh.close()
    used.close()
