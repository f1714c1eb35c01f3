"""Rounding error of the float32 GEMMs against float64 (needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.binding import Engine
from paper_2412_18910_amd.config import FP32, Config

from .gpu_helpers import to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1024, 2048, 4096, 8192])   # 8 waves in the decode GEMM; both chain lengths of the prompt GEMM
@pytest.mark.parametrize("sign", ["both", "one"])   # of one sign: a rounding that leans one way would add up
def test_sums_lose_no_more_than_scalar_sums(k, sign):
    """V rows of the first layer (normalised embedding times wv), by the prompt pass and by a verification block.

    A wave of scalar code sums K products as 64 chains of K / 64 and a butterfly of 6 levels: K / 128 + 6 roundings at
    the result's magnitude, two more for its normalised input.  A rounding is 0.42 * 2^-24 of a value in the mean
    (uniform error, mantissas log-uniform), 0.5 leaves a sixth.  One chain per accumulator costs K / 64 and more."""
    cfg = Config(1, k, 4, 4, 64, 64, 64, dtype=FP32, k_max=7, n_ctx_max=128, ldlp_hidden=64)
    w = synth.make_weights(cfg, 91)
    if sign == "one":
        w["tok_emb"].abs_()
        w["layers"][0]["wv"].abs_()
    eng = Engine(cfg, to_device(w))
    ids = synth.token_ids(60, cfg.vocab, 92)
    block = synth.token_ids(8, cfg.vocab, 93)
    eng.prefill(ids)      # more than 16 tokens: the prompt GEMMs
    eng.verify(block)
    x = w["tok_emb"][torch.as_tensor(np.concatenate([ids, block]), dtype=torch.long)].double()
    y = x / torch.sqrt((x * x).mean(-1, keepdim=True) + cfg.rms_eps) * w["layers"][0]["attn_norm"].double()
    v = (y @ w["layers"][0]["wv"].double().T).numpy()
    bound = 0.5 * 2.0 ** -24 * np.sqrt(k / 128 + 8)
    for part in (slice(0, 60), slice(60, 68)):
        got = np.stack([eng.kv_row(0, 1, s) for s in range(part.start, part.stop)]).astype(np.float64)
        err = np.linalg.norm(got - v[part]) / np.linalg.norm(v[part])
        print(f"K {k} rows {part.start}..{part.stop - 1}: {err:.3e} of {bound:.3e}")
        assert err <= bound, (part, err, bound)
    eng.close()
