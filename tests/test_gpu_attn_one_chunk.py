"""Contexts that one attention workgroup holds whole, at the edge to two of them (needs an MI355X)."""
import numpy as np
import pytest

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.config import BF16, FP32, Config

from .gpu_helpers import make_pair

pytestmark = pytest.mark.gpu

TOL = {FP32: 1e-4, BF16: 2e-2}


def _cfg(dtype, hd):
    return Config(2, 256, 8, 2, hd, 512, 1008, dtype=dtype, k_max=5, n_ctx_max=320, ldlp_hidden=64)


@pytest.mark.parametrize("dtype,hd,edge", [(BF16, 64, 256), (BF16, 128, 256), (FP32, 64, 64), (FP32, 128, 64)])
@pytest.mark.parametrize("before", [1, 3, 6])
def test_blocks_around_the_edge(dtype, hd, edge, before):
    """Rows that see up to `edge` slots in a block that ends before, at or behind it: as the oracle has them, and bit
    for bit alike in every such block (a second workgroup whose slots a row does not see has weight 0)."""
    cfg = _cfg(dtype, hd)
    eng, orc, _ = make_pair(cfg, 61)
    n = edge - before
    ids = synth.token_ids(n, cfg.vocab, 62)
    block = synth.token_ids(6, cfg.vocab, 63)
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
                assert np.max(np.abs(orc.logits(r) - lg)) <= TOL[dtype], (rows, r)
            assert np.array_equal(first[r], lg), (rows, r)
    eng.close()
