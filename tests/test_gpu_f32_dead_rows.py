"""Float32: cache rows behind the end of a block, rolled back or left by an earlier sequence, may hold anything (needs an
MI355X)."""
import numpy as np
import pytest

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.binding import Engine
from paper_2412_18910_amd.config import FP32, Config

from .gpu_helpers import to_device

pytestmark = pytest.mark.gpu

NAN, INF = 7, 11   # tokens whose embedding is not finite
CFG = {64: Config(2, 264, 4, 2, 64, 712, 1003, dtype=FP32, k_max=7, n_ctx_max=320, ldlp_hidden=64),
       128: Config(2, 256, 4, 1, 128, 512, 1000, dtype=FP32, k_max=7, n_ctx_max=320, ldlp_hidden=64)}


@pytest.fixture(params=[64, 128])
def eng(request):
    cfg = CFG[request.param]
    w = synth.make_weights(cfg, 95)
    w["tok_emb"][NAN] = float("nan")
    w["tok_emb"][INF] = float("inf")
    e = Engine(cfg, to_device(w))
    yield e
    e.close()


def _ids(eng, n):
    ids = synth.token_ids(n, eng.cfg.vocab, 96)
    ids[(ids == NAN) | (ids == INF)] = 20
    return ids


@pytest.mark.parametrize("n", [5, 15, 16, 61, 64, 200])
def test_rolled_back_rows(eng, n):
    """Blocks behind n slots, at every place in a tile of 16 keys and a chunk of 64."""
    eng.prefill(_ids(eng, n))
    good = np.array([20, 21], np.int32)
    eng.verify(good)
    clean = [eng.logits(i) for i in range(2)]
    assert all(np.isfinite(x).all() for x in clean)
    eng.verify(np.array([20, 21, NAN, INF, NAN, INF], np.int32))
    assert not np.isfinite(eng.logits(5)).all()
    eng.verify(good)
    for i in range(2):
        assert np.array_equal(eng.logits(i), clean[i]), i


@pytest.mark.parametrize("n", [9, 20, 33, 77, 130])
@pytest.mark.parametrize("mode", [Engine.PREFILL_AUTO, Engine.PREFILL_BLOCKS])
def test_rows_of_an_earlier_prompt(eng, n, mode):
    eng.set_prefill_mode(mode, 128)   # 130: a chunk of two rows
    ids = _ids(eng, n)
    eng.prefill(ids)
    clean = eng.logits(0), eng.kv_row(1, 1, n - 1), eng.kv_row(2, 0, n - 2)
    assert np.isfinite(clean[0]).all()
    eng.prefill(np.concatenate([ids, np.full(40, NAN, np.int32)]))
    eng.prefill(ids)
    for a, b in zip(clean, (eng.logits(0), eng.kv_row(1, 1, n - 1), eng.kv_row(2, 0, n - 2))):
        assert np.array_equal(a, b)


def test_a_feature_that_is_not_finite_spoils_its_own_slot_only(eng):
    n = 40
    eng.prefill(_ids(eng, n))
    feat = eng.feature((n - 1) % 16)
    bad = np.full(eng.cfg.d_model, np.nan, np.float32)

    def drafted(slots):
        eng.set_state(slots, 20, 21, feat)
        eng.draft(2, override_ids=np.array([20, 21], np.int32))
        return [eng.draft_logits(i) for i in range(2)]

    clean = drafted(n - 2)
    eng.set_state(n, 20, 21, bad)
    eng.draft(3, override_ids=np.array([20, 21, 20], np.int32))
    for a, b in zip(clean, drafted(n - 2)):
        assert np.isfinite(a).all() and np.array_equal(a, b)
