"""Rows fetched in any order, between steps, while earlier ones are kept (needs an MI355X)."""
import numpy as np
import pytest

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.binding import Engine
from paper_2412_18910_amd.config import BF16, FP32, Config

from .gpu_helpers import to_device

pytestmark = pytest.mark.gpu


# rows shorter than a piece of 4096, of one piece and a bit (unaligned in the odd vocabulary), of several
@pytest.mark.parametrize("dtype,vocab", [(BF16, 512), (FP32, 4099), (BF16, 20480)])
def test_rows_in_any_order(dtype, vocab):
    cfg = Config(1, 256, 4, 2, 64, 512, vocab, dtype=dtype, k_max=6, n_ctx_max=128, ldlp_hidden=64)
    eng = Engine(cfg, to_device(synth.make_weights(cfg, 31)))
    ids = synth.token_ids(20, vocab, 32)
    eng.prefill(ids)
    feat, pending = eng.feature(19 % 16), eng.pending
    rng, kept = np.random.default_rng(33), []
    for trial in range(8):
        block = synth.token_ids(7, vocab, 40 + trial)
        eng.set_state(20, int(ids[-1]), pending, feat)
        eng.draft(6, override_ids=block[1:])
        eng.verify(block)
        alone = []
        for i in range(7):      # each behind another fetch: never sent ahead
            eng.feature(0)
            alone.append((eng.logits(i).copy(), eng.draft_logits(min(i, 5)).copy()))
        assert not np.array_equal(alone[0][0], alone[1][0])
        order = range(7) if trial < 2 else rng.integers(0, 7, 30)
        for i in order:
            row = eng.logits(i)
            assert np.array_equal(row, alone[i][0])
            kept.append((row, alone[i][0]))
            if trial % 2:
                assert np.array_equal(eng.draft_logits(min(i, 5)), alone[i][1])
        for i in range(6):
            assert np.array_equal(eng.draft_logits(i), alone[i][1])
        eng.logits(0), eng.logits(1)   # row 2 is on its way when the next block is verified
        if trial == 4:
            kept = kept[::3]
    assert all(np.array_equal(a, b) for a, b in kept)
    eng.close()
