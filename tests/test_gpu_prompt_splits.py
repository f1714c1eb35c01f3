"""bf16 prompts whose GEMMs split K over workgroups, at the edges of the row tiles (needs an MI355X)."""
import numpy as np
import pytest

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.binding import Engine
from paper_2412_18910_amd.config import BF16, Config

from .gpu_helpers import make_pair, to_device
from .test_gpu_dense_prefill import TOL, check_state, steps_after

pytestmark = pytest.mark.gpu

# K of 1024 and 2816 (pieces of unequal length), output widths that are no multiple of the 128-row tile
MID = Config(2, 1024, 8, 2, 64, 2816, 2000, dtype=BF16, k_max=5, n_ctx_max=768, ldlp_hidden=64)


@pytest.mark.parametrize("n,chunk", [(17, 0), (63, 0), (64, 0), (65, 0), (128, 0), (129, 0), (257, 128)])
def test_prompt_state_matches_oracle(n, chunk):
    eng, orc, _ = make_pair(MID, 51)
    ids = synth.token_ids(n, MID.vocab, 700 + n)
    orc.prefill(ids)
    eng.set_prefill_mode(Engine.PREFILL_AUTO, chunk)
    eng.prefill(ids)
    check_state(MID, eng, orc, n, slots=sorted({0, 15, 16, n - 2, n - 1}))
    steps_after(MID, eng, orc, 2)
    eng.close()


@pytest.mark.parametrize("bias", [True, False])
def test_prompt_passes_agree_with_and_without_a_draft_bias(bias):
    w = to_device(synth.make_weights(MID, 52))
    if not bias:
        w["draft_fc_b"] = None
    eng = Engine(MID, w)
    ids = synth.token_ids(700, MID.vocab, 5)
    out = []
    for mode in (Engine.PREFILL_BLOCKS, Engine.PREFILL_DENSE):
        eng.set_prefill_mode(mode, 0)
        eng.prefill(ids)
        out.append((eng.logits(0), eng.kv_row(MID.n_layers, 0, 698), eng.kv_row(MID.n_layers, 1, 3)))
    (lb, kb, vb), (ld, kd, vd) = out
    assert np.max(np.abs(lb - ld)) <= TOL
    for a, b in ((kb, kd), (vb, vd)):   # a flipped bf16 rounding is 2^-8 of an element
        assert np.max(np.abs(a - b)) <= np.max(np.abs(a)) * 2 ** -7
    eng.close()
