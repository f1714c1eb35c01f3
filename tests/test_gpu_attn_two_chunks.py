"""Contexts that one attention workgroup holds as two chunks, at the edges to one and to three of them (needs an MI355X)."""
import numpy as np
import pytest

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.config import BF16, FP32, Config

from .gpu_helpers import make_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,hd,kv,edge", [(BF16, 64, 4, 256), (BF16, 128, 4, 256), (BF16, 128, 2, 256), (FP32, 64, 2, 64), (FP32, 128, 4, 64)])
@pytest.mark.parametrize("chunks,before", [(1, 3), (2, 6), (2, 3)])
def test_rows_do_not_depend_on_the_block(dtype, hd, kv, edge, chunks, before):
    """Blocks of 1 to 6 rows that end before, at or behind the edge, with one or (grouped queries, bf16) two tiles of rows: rows as the
    oracle has them, and bit for bit alike whether one workgroup or a merge launch has put their chunks together."""
    cfg = Config(2, 256, 4 if kv == 4 else 8, kv, hd, 512, 1008, dtype=dtype, k_max=5, n_ctx_max=600, ldlp_hidden=64)
    eng, orc, _ = make_pair(cfg, 71)
    n = chunks * edge - before
    ids = synth.token_ids(n, cfg.vocab, 72)
    block = synth.token_ids(6, cfg.vocab, 73)
    orc.prefill(ids)
    eng.prefill(ids)
    orc.verify(block)
    first = {}
    for rows in range(1, 7):
        eng.verify(block[:rows])
        for r in range(rows):
            lg = eng.logits(r)
            if r not in first:
                first[r] = lg
                assert np.max(np.abs(orc.logits(r) - lg)) <= (1e-4 if dtype == FP32 else 2e-2), (rows, r)   # the parity tests' bars
            assert np.array_equal(first[r], lg), (rows, r)
    eng.close()
