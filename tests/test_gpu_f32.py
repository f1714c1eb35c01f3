"""Float32 models on the GPU against the oracle at the sizes where the kernels change shape (needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.binding import Engine
from paper_2412_18910_amd.config import FP32, Config

from .gpu_helpers import make_pair, to_device, top2_margin

pytestmark = pytest.mark.gpu

TOL = 1e-4      # the float32 bar of the parity tests: logits of order one, sums of a few thousand terms
# widths that are multiples of 8 only (half row-blocks, K tails), an odd vocabulary, grouped queries
RAGGED = Config(2, 264, 4, 2, 64, 712, 1003, dtype=FP32, k_max=7, n_ctx_max=768, ldlp_hidden=64)
# head_dim 128, K of 1024 and more (8 waves per workgroup), more query rows than one tile of 16 per KV head
WIDE = Config(1, 1032, 8, 2, 128, 1544, 2048, dtype=FP32, k_max=9, n_ctx_max=512, ldlp_hidden=64)


def same_state(cfg, eng, orc, n):
    lo, lg = orc.logits(0), eng.logits(0)
    assert np.max(np.abs(lo - lg)) <= TOL, float(np.max(np.abs(lo - lg)))
    if top2_margin(lo) > 2 * TOL:
        assert eng.pending == orc.pending
    assert np.max(np.abs(orc.feature((n - 1) % (cfg.k_max + 1)) - eng.feature((n - 1) % 16))) <= TOL
    for layer in (0, cfg.n_layers):
        for which in (0, 1):
            for slot in {0, 16 % n, n // 2, n - 2}:
                a, b = orc.kv_row(layer, which, slot), eng.kv_row(layer, which, slot)
                assert np.max(np.abs(a - b)) <= TOL, (layer, which, slot)


def one_step(cfg, eng, orc, k):
    d = orc.draft(k)
    assert np.array_equal(d, eng.draft(k, override_ids=d))
    for i in range(k):
        assert np.max(np.abs(orc.draft_logits(i) - eng.draft_logits(i))) <= TOL * max(1.0, float(np.std(orc.draft_logits(i)))), i
    orc.verify(n_rows=k + 1)
    eng.verify(n_rows=k + 1)
    for i in range(k + 1):
        assert np.max(np.abs(orc.logits(i) - eng.logits(i))) <= TOL, i
    return orc.accept() == eng.accept()


@pytest.mark.parametrize("cfg", [RAGGED, WIDE], ids=["ragged-hd64", "wide-hd128"])
@pytest.mark.parametrize("n,chunk", [(17, 0), (32, 0), (33, 0), (64, 0), (65, 0), (130, 128), (257, 128), (300, 0)])
def test_prompt_and_steps_match_oracle(cfg, n, chunk):
    """Prompts around the multiples of 16, 32 and 64 rows, in one chunk and in several (a one-row last chunk among
    them).  These widths take tiles of 16 rows nearly everywhere; the other tiles: test_gpu_prompt_tiles.py."""
    eng, orc, _ = make_pair(cfg, 41)
    ids = synth.token_ids(n, cfg.vocab, 900 + n)
    orc.prefill(ids)
    eng.set_prefill_mode(Engine.PREFILL_AUTO, chunk)
    eng.prefill(ids)
    same_state(cfg, eng, orc, n)
    for k in (1, cfg.k_max):
        if not one_step(cfg, eng, orc, k):
            break   # a sub-margin row
    eng.close()


def test_prompt_passes_agree_and_short_prompts_keep_the_block_pass():
    eng, _, _ = make_pair(RAGGED, 42)
    ids = synth.token_ids(500, RAGGED.vocab, 5)
    out = {}
    for mode in (Engine.PREFILL_BLOCKS, Engine.PREFILL_AUTO):
        eng.set_prefill_mode(mode)
        eng.prefill(ids)
        long = eng.logits(0), eng.kv_row(RAGGED.n_layers, 1, 498)
        eng.prefill(ids[:16])
        out[mode] = long + (eng.logits(0),)
    b, a = out[Engine.PREFILL_BLOCKS], out[Engine.PREFILL_AUTO]
    assert np.max(np.abs(a[0] - b[0])) <= TOL and np.max(np.abs(a[1] - b[1])) <= TOL
    assert np.array_equal(a[2], b[2])
    eng.close()


@pytest.mark.parametrize("n_ctx", [1, 15, 63, 64, 65, 255, 300])
def test_block_equals_single_rows_bit_exact_across_chunk_edges(n_ctx):
    """A block's rows must not depend on the rows beside them, wherever its slots fall among the 64-key chunks."""
    eng, _, _ = make_pair(RAGGED, 43)
    ids = synth.token_ids(n_ctx, RAGGED.vocab, 6)
    block = synth.token_ids(RAGGED.k_max + 1, RAGGED.vocab, 7)
    eng.prefill(ids)
    eng.verify(block)
    whole = [eng.logits(i) for i in range(len(block))]
    eng.prefill(ids)
    for i, t in enumerate(block):
        eng.verify([int(t)])
        assert np.array_equal(whole[i], eng.logits(0)), i
        eng.accept()
    eng.close()


def test_sampled_draft_and_ddd_statistic_with_an_odd_vocabulary():
    """LM head without argmax partials (a sampled token) and with softmax partials (the exit rule)."""
    cfg = RAGGED.with_(temperature=0.7, ddd_enabled=1, ddd_threshold=-1e9)
    for c in (RAGGED.with_(temperature=0.7), cfg):
        eng, orc, _ = make_pair(c, 44)
        ids = synth.token_ids(40, c.vocab, 8)
        orc.prefill(ids)
        eng.prefill(ids)
        u = synth.uniforms(c.k_max, 9)
        d_o, d_g = orc.draft(3, u_draft=u), eng.draft(3, u_draft=u)
        assert np.array_equal(d_o, d_g)
        if c.ddd_enabled:
            assert len(d_g) == c.k_max
            assert abs(eng.draft_logprob - sum(
                float(l[t] / 0.7 - np.log(np.sum(np.exp(l.astype(np.float64) / 0.7))))
                for l, t in ((eng.draft_logits(i), d_g[i]) for i in range(c.k_max)))) < 1e-3
        eng.close()


def test_weights_that_begin_at_any_float():
    """Matrices are contiguous, but may begin anywhere in a larger tensor: the same bits from every alignment."""
    cfg = Config(2, 264, 4, 2, 64, 520, 515, dtype=FP32, k_max=4, n_ctx_max=128, ldlp_hidden=64)
    w = synth.make_weights(cfg, 71)
    ids, block = synth.token_ids(70, cfg.vocab, 72), synth.token_ids(5, cfg.vocab, 73)

    def moved(t, by):
        if t is None or t.dim() < 2:
            return t
        store = torch.empty(t.numel() + by, dtype=t.dtype, device="cuda")
        store[by:].copy_(t.reshape(-1))
        return store[by:].view(t.shape)

    def run(by):
        dev = {k: moved(v, by) if torch.is_tensor(v) else v for k, v in to_device(w).items()}
        dev["layers"] = [{k: moved(v, by) for k, v in lw.items()} for lw in dev["layers"]]
        dev["draft_layer"] = {k: moved(v, by) for k, v in dev["draft_layer"].items()}
        eng = Engine(cfg, dev)
        eng.prefill(ids)
        out = [eng.logits(0)]
        d = eng.draft(4)
        eng.verify(block)
        out += [eng.logits(i) for i in range(5)] + [eng.draft_logits(i) for i in range(4)] + [d]
        eng.close()
        return out

    want = run(0)
    for by in (1, 2, 3):
        assert all(np.array_equal(a, b) for a, b in zip(want, run(by)))
