"""Prompts at widths where the layout of a prompt GEMM goes by its estimated time: every row-block count of a tile, whole K and
pieces of it, ragged row counts (needs an MI355X).  tests/test_host_prompt_plans.py checks which kernels each case reaches."""
import numpy as np
import pytest

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.binding import Engine
from paper_2412_18910_amd.config import BF16, FP32, Config

from .gpu_helpers import to_device
from .test_gpu_prompt_tiles import compare, rows_of

pytestmark = pytest.mark.gpu


def _cfg(d, heads, kv, ffn, hd=64, dtype=BF16):
    return Config(1, d, heads, kv, hd, ffn, 512, dtype=dtype, k_max=5, n_ctx_max=2600, ldlp_hidden=64)


# bf16: (widths), rows, (epilogue, row-blocks of a tile, weight row-blocks of a wave, waves); the widths end within tiles of 8, 12, 16, 24
# and 32 weight row-blocks; RESID over 1743 and 2133 rows: the last tile reaches behind the buffers
CASES = [
    ((768, 8, 8, 4096), 20, {("PART", 2, 2, 4)}),
    ((3072, 16, 16, 6144), 37, {("PART", 3, 2, 4), ("PART", 3, 3, 4), ("PART", 4, 2, 8)}),
    ((3072, 16, 16, 6144), 61, {("PART", 4, 2, 4), ("PART", 4, 3, 4)}),
    ((4352, 8, 8, 4352), 141, {("PART", 5, 2, 4), ("PART", 5, 2, 8), ("PART", 5, 3, 4)}),
    ((4352, 8, 8, 4352), 173, {("PART", 6, 2, 4), ("PART", 6, 2, 8), ("PART", 6, 3, 4)}),
    ((3072, 8, 8, 3072), 300, {("PART", 7, 2, 4), ("PART", 7, 2, 8), ("PART", 7, 3, 4)}),
    ((3072, 8, 8, 3072), 365, {("SWIGLU", 4, 2, 8)}),
    ((3072, 16, 16, 6144), 501, {("SWIGLU", 7, 2, 8)}),
    ((3072, 48, 16, 4096), 701, {("QKV", 5, 2, 8), ("SWIGLU", 6, 2, 8)}),
    ((4096, 4, 2, 4096), 701, {("RESID", 4, 2, 8)}),
    ((4352, 8, 8, 4352), 901, {("SWIGLU", 5, 4, 8)}),
    ((3072, 48, 16, 4096), 1001, {("QKV", 6, 2, 8), ("SWIGLU", 8, 2, 8)}),
    ((4096, 4, 2, 4096), 1101, {("PART", 8, 2, 4), ("PART", 8, 2, 8), ("PART", 8, 3, 4), ("RESID", 5, 2, 8), ("SWIGLU", 5, 2, 8)}),
    ((3072, 8, 8, 3072), 1743, {("QKV", 4, 2, 8), ("RESID", 6, 2, 8), ("SWIGLU", 6, 4, 8)}),
    ((3072, 32, 8, 3072), 2133, {("QKV", 7, 2, 8), ("RESID", 7, 2, 8), ("SWIGLU", 7, 4, 8)}),
    ((3072, 32, 8, 3072), 2501, {("QKV", 8, 2, 8), ("RESID", 8, 2, 8), ("SWIGLU", 8, 4, 8)}),
]

# float32, widths of whole tiles: (epilogue, row-blocks of a tile, long chains) or ("TAIL-" epilogue, row-blocks, behind whole tiles).  K = 64
# is three stages, K of 128 and 1024 six and 33: the loop's remainder.
CASES += [
    ((64, 4, 4, 2048, 64, FP32), 133, {("SWIGLU", 2, 0)}),
    ((64, 4, 4, 2048, 64, FP32), 403, {("SWIGLU", 4, 0)}),
    ((4096, 8, 8, 1024, 128, FP32), 37, {("PART", 3, 1), ("QKV", 3, 1), ("SWIGLU", 2, 1), ("TAIL-QKV", 3, 0), ("TAIL-SWIGLU", 2, 0)}),
    ((4096, 8, 8, 1024, 128, FP32), 61, {("PART", 4, 1), ("QKV", 4, 1), ("TAIL-QKV", 4, 0)}),
    ((4096, 8, 8, 1024, 128, FP32), 101, {("PART", 4, 0), ("SWIGLU", 4, 1), ("TAIL-SWIGLU", 4, 0)}),
    ((4096, 8, 8, 1024, 128, FP32), 2001, {("TAIL-QKV", 4, 1)}),
]


@pytest.mark.parametrize("widths,n,_", CASES, ids=["%s%d-%d-%d" % ("f32-" if FP32 in c[0][4:] else "", c[0][0], c[0][3], c[1]) for c in CASES])
def test_every_row_against_the_16_row_pass(widths, n, _):
    cfg = _cfg(*widths)
    eng = Engine(cfg, to_device(synth.make_weights(cfg, 111)))
    ids = synth.token_ids(n, cfg.vocab, 112)
    slots = list(range(n - 1))
    got = []
    for mode in (Engine.PREFILL_BLOCKS, Engine.PREFILL_AUTO):
        eng.set_prefill_mode(mode, 8192)   # one chunk
        eng.prefill(ids)
        got.append((eng.logits(0), rows_of(eng, cfg, slots)))
    eng.close()
    assert np.max(np.abs(got[0][0] - got[1][0])) <= (1e-4 if cfg.dtype == FP32 else 2e-2)   # the bars of the parity tests
    compare(cfg, got[0][1], got[1][1])
