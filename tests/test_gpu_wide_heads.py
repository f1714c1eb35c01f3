"""LM heads of vocabularies that take 16 row-blocks a workgroup, ragged and whole, one k-tile a wave and several (needs an MI355X)."""
import numpy as np
import pytest

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.config import BF16, Config

from .gpu_helpers import make_pair
from .test_gpu_dense_prefill import TOL

pytestmark = pytest.mark.gpu


# 2501 row-blocks (the last workgroup slides back over 11 of its neighbour's), 4096 (one whole round), 8016 (two)
@pytest.mark.parametrize("d,heads,vocab,rows", [(256, 4, 40016, 1), (768, 4, 40016, 6), (256, 4, 65536, 5), (256, 4, 128256, 6)])
def test_logits_argmax_and_draft_probability(d, heads, vocab, rows):
    cfg = Config(1, d, heads, 2, 64, 256, vocab, dtype=BF16, k_max=5, n_ctx_max=64, ldlp_hidden=64, ddd_enabled=1, ddd_threshold=-1e9)
    eng, orc, _ = make_pair(cfg, 61)
    ids = synth.token_ids(20, vocab, 62)
    orc.prefill(ids)
    eng.prefill(ids)
    block = synth.token_ids(rows, vocab, 63)
    orc.verify(block)
    eng.verify(block)
    got = np.stack([eng.logits(i) for i in range(rows)])
    assert np.max(np.abs(got - np.stack([orc.logits(i) for i in range(rows)]))) <= TOL
    accepted, bonus = eng.accept()
    assert bonus == eng.pending == int(np.argmax(got[accepted]))
    # a block whose drafts are the argmaxes of the rows before them: each row's own argmax, over all workgroups, is asked for
    eng.prefill(ids)
    block = block[:1]
    while len(block) < rows:
        eng.verify(block)
        block = np.append(block, np.argmax(eng.logits(len(block) - 1))).astype(np.int32)
    eng.verify(block)
    got = np.stack([eng.logits(i) for i in range(rows)])
    assert eng.accept() == (rows - 1, int(np.argmax(got[-1])))
    assert np.array_equal(block[1:], got[:-1].argmax(1))
    eng.prefill(ids)
    draft = eng.draft(3)
    logits = np.stack([eng.draft_logits(i) for i in range(len(draft))]).astype(np.float64)
    assert np.array_equal(draft, logits.argmax(1))
    logp = sum(l[t] - l.max() - np.log(np.exp(l - l.max()).sum()) for l, t in zip(logits, draft))
    assert abs(eng.draft_logprob - logp) <= 1e-5 * len(draft) * max(1.0, abs(logp))   # float32 sums of exponentials
    eng.close()
