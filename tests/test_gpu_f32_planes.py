"""Float32 prompts on the bf16 matrix instruction: three bf16 parts a number (needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.binding import Engine
from paper_2412_18910_amd.config import FP32, Config

from .gpu_helpers import to_device

pytestmark = pytest.mark.gpu

N = 50


def rows_of_both_passes(cfg, w, n=N):
    """K and V rows of the first layer by the 16-row pass of the decode kernels and by the prompt pass."""
    eng = Engine(cfg, to_device(w))
    ids = np.arange(n, dtype=np.int32) % cfg.vocab
    out = []
    for mode in (Engine.PREFILL_BLOCKS, Engine.PREFILL_AUTO):
        eng.set_prefill_mode(mode)
        eng.prefill(ids)
        out.append(np.stack([[eng.kv_row(0, which, s) for which in (0, 1)] for s in range(n - 1)]))
    eng.close()
    return out


# tails of a k-tile (8, 16, 24), a single k-tile, thrice as many k-tiles as the shortest loop and one more
@pytest.mark.parametrize("d", [8, 32, 72, 96, 104, 272, 1032])
def test_tails_of_k(d):
    cfg = Config(1, d, 4, 2, 64, 24, 64, dtype=FP32, k_max=3, n_ctx_max=64, ldlp_hidden=64)
    a, b = rows_of_both_passes(cfg, synth.make_weights(cfg, 11))
    # two correct sums of d products differ by a few roundings of the largest partial sums, 2^-24 each
    assert np.max(np.abs(a - b)) <= 2.0 ** -24 * 64 * np.max(np.abs(a))


# exponents of the normalised activations and of the weights: their products stay ordinary numbers
@pytest.mark.parametrize("ex,ew", [(0, 0), (60, -107), (85, -120), (90, -130), (-105, 40), (-118, 60), (-140, 95), (-50, -50)])
def test_small_numbers_keep_their_bits(ex, ew):
    """K and V rows of the first layer where one side of all products is so small that bf16 has no numbers for its last bits
    (below 2^-110), or where it is a float32 subnormal.  The bound is that of the scalar sums (test_gpu_f32_error.py)."""
    d = 1024
    cfg = Config(1, d, 4, 4, 64, 64, 64, dtype=FP32, k_max=3, n_ctx_max=64, ldlp_hidden=64)
    w = synth.make_weights(cfg, 13)
    lw = w["layers"][0]
    lw["attn_norm"] = (lw["attn_norm"].double() * 2.0 ** ex).float()
    for name in ("wk", "wv"):
        lw[name] = (lw[name].double() * 2.0 ** ew).float()
    lw["wq"].zero_()   # (scores: nothing of the kind matters here)
    x = w["tok_emb"].double()
    y = (x / torch.sqrt((x * x).mean(-1, keepdim=True) + cfg.rms_eps) * lw["attn_norm"].double())[:N - 1]
    want = (y @ lw["wv"].double().T).numpy()
    a, b = rows_of_both_passes(cfg, w)
    bound = 0.5 * 2.0 ** -24 * np.sqrt(d / 128 + 8)
    if ex < -125:   # the activations are subnormal numbers themselves: each is rounded to a multiple of 2^-149
        bound += 0.5 * 2.0 ** -149 / float(y.abs().mean())
    errs = [float(np.linalg.norm(r[:, 1] - want) / np.linalg.norm(want)) for r in (a, b)]
    print(ex, ew, errs, bound)
    assert errs[1] <= bound
    assert np.linalg.norm(a[:, 0] - b[:, 0]) <= (errs[0] + 2 * bound) * np.linalg.norm(a[:, 0])


def test_numbers_at_the_ends_of_the_range():
    """Weights and normalised activations between the largest bf16 and the largest float, tiny ones beside them, Inf and NaN."""
    cfg = Config(1, 128, 4, 2, 64, 64, 64, dtype=FP32, k_max=3, n_ctx_max=64, ldlp_hidden=64)
    w = synth.make_weights(cfg, 12)
    lw = w["layers"][0]
    emb = torch.where(torch.arange(128) % 3 == 0, -1.0, 1.0).repeat(64, 1) * (1 + 0.001 * torch.randn(64, 128, generator=torch.Generator().manual_seed(3)))
    emb[:, 5] = 1.0
    w["tok_emb"] = emb.float().contiguous()
    lw["attn_norm"][5] = 3.396e38   # times one: a float that rounds to Inf in bf16
    lw["attn_norm"][6] = 1e-38      # (its products are of order one, as those of column 5 and all others together)
    for name in ("wq", "wk", "wv"):
        lw[name][:, 5] = 3e-39 * torch.randn(lw[name].shape[0], generator=torch.Generator().manual_seed(4))
        lw[name][:, 6] = 3.397e38 * (1 if name == "wv" else -1)
    x = w["tok_emb"].double()
    y = x / torch.sqrt((x * x).mean(-1, keepdim=True) + cfg.rms_eps) * lw["attn_norm"].double()
    want = (y @ lw["wv"].double().T).numpy()
    a, b = rows_of_both_passes(cfg, w)
    assert np.isfinite(a).all() and np.isfinite(b).all()
    assert np.max(np.abs(want)) < 20   # the small numbers' products would be seen if they were missing
    # what is normalised in another order differs by the last bit of a subnormal number, 2^-23 of 1e-38
    for got in (a, b):
        assert np.max(np.abs(got[:, 1] - want[:N - 1])) <= 2.0 ** -20 * np.max(np.abs(want))
    # an Inf, a NaN and a sum that overflows stay where they are
    w["tok_emb"][7, 9] = float("inf")
    w["tok_emb"][20, 3] = float("nan")
    lw["wv"][3, 5] = 2.0
    lw["wv"][70, 40] = float("-inf")
    a, b = rows_of_both_passes(cfg, w)
    assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isposinf(a), np.isposinf(b)) and \
        np.array_equal(np.isneginf(a), np.isneginf(b))
    ok = np.isfinite(a)
    assert ok.mean() > 0.9 and np.max(np.abs(a[ok] - b[ok])) <= 2.0 ** -19 * np.max(np.abs(want))   # 2^-20 on either side
