"""Causal attention of prompt chunks whose waves own one or two tiles of query rows (needs an MI355X)."""
import numpy as np
import pytest

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.binding import Engine
from paper_2412_18910_amd.config import BF16, Config

from .gpu_helpers import to_device
from .test_gpu_dense_prefill import TOL

pytestmark = pytest.mark.gpu


# chunks of 1536 rows: the first has no context (one tile a wave), the second has as many slots before it as rows and
# 384 workgroups of two tiles a wave, the last is ragged (two tiles a wave from 1536 rows on, one below)
@pytest.mark.parametrize("heads,kv,hd,n", [(32, 8, 64, 3072), (32, 8, 128, 3079), (32, 32, 64, 4607)])
def test_dense_chunks_agree_with_blocks(heads, kv, hd, n):
    cfg = Config(1, 256, heads, kv, hd, 512, 1008, dtype=BF16, k_max=4, n_ctx_max=n + 16, ldlp_hidden=64)
    eng = Engine(cfg, to_device(synth.make_weights(cfg, 55)))
    ids = synth.token_ids(n, cfg.vocab, 56)
    out = []
    for mode in (Engine.PREFILL_BLOCKS, Engine.PREFILL_DENSE):
        eng.set_prefill_mode(mode, 1536)
        eng.prefill(ids)
        rows = [eng.kv_row(1, w, s) for w in (0, 1) for s in (0, 1535, 1536, 2000, n - 2)]   # draft head: behind attention
        out.append((eng.logits(0), rows))
    (lb, kb), (ld, kd) = out
    assert np.max(np.abs(lb - ld)) <= TOL
    for a, b in zip(kb, kd):   # a flipped bf16 rounding is 2^-8 of an element
        assert np.max(np.abs(a - b)) <= np.max(np.abs(a)) * 2 ** -7
    eng.close()
