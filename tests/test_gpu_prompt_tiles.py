"""Prompts that reach every tile shape of the prompt GEMMs, at ragged row counts (needs an MI355X).

The rules that choose a tile go by the number of tiles, so each case names the kernels it is there for; tests/
test_host_prompt_tiles.py checks that it still reaches them.  The prompt pass is compared row by row with the 16-row
pass of the decode kernels, and where the oracle is quick enough with the oracle."""
from dataclasses import dataclass

import numpy as np
import pytest

from paper_2412_18910_amd import synth
from paper_2412_18910_amd.binding import Engine
from paper_2412_18910_amd.config import BF16, FP32, Config

from .gpu_helpers import make_pair, to_device

pytestmark = pytest.mark.gpu


def _cfg(dtype, d, heads, kv, hd, ffn):
    return Config(1, d, heads, kv, hd, ffn, 515 if dtype == FP32 else 512, dtype=dtype, k_max=5, ldlp_hidden=64)


@dataclass(frozen=True)
class Case:
    cfg: Config
    n: int
    reaches: tuple
    oracle: bool = True
    chunk: int = 0

    @property
    def config(self):
        return self.cfg.with_(n_ctx_max=self.n + 16)


# float32: (epilogue, 16-row blocks of a tile, long chains), ("TAIL-" epilogue, 16-row blocks of a tile, 1: behind whole tiles)
# where the last tiles are made in pieces of K; widths leave tails in K and half row-blocks
F_SHORT, F_LONG = _cfg(FP32, 1032, 16, 8, 128, 4104), _cfg(FP32, 4104, 16, 8, 128, 4104)
F_MID, F_2K, F_MHA = _cfg(FP32, 1032, 12, 6, 64, 2056), _cfg(FP32, 2056, 16, 8, 128, 4104), _cfg(FP32, 1032, 32, 32, 128, 4104)
F_WIDE = _cfg(FP32, 4104, 32, 8, 128, 1032)
# bf16, whole K: (epilogue, row-blocks of a tile, weight row-blocks of a wave, waves); the widths of QKV (120 and 264 row-blocks)
# and of B_ODD (272) end within a tile of 16, those of B_ODD within one of 32
B_FFN, B_WIDE, B_QKV = _cfg(BF16, 256, 4, 2, 64, 4096), _cfg(BF16, 4096, 4, 4, 64, 256), _cfg(BF16, 256, 20, 5, 64, 512)
B_QKV2, B_ODD = _cfg(BF16, 256, 44, 11, 64, 4352), _cfg(BF16, 4352, 4, 4, 64, 256)
# bf16, K in pieces
B_SPLIT = _cfg(BF16, 1024, 4, 2, 64, 11008)
CASES = {
    "f32-61": Case(F_SHORT, 61, (("PART", 1, 0), ("QKV", 1, 0), ("SWIGLU", 2, 0), ("PART", 1, 1), ("TAIL-QKV", 1, 0))),
    "f32-101": Case(F_MID, 101, (("PART", 1, 0), ("QKV", 1, 0), ("SWIGLU", 1, 0), ("TAIL-SWIGLU", 1, 0))),
    "f32-131": Case(F_SHORT, 131, (("QKV", 2, 0), ("SWIGLU", 3, 0), ("TAIL-QKV", 2, 0))),
    "f32-163": Case(F_SHORT, 163, (("TAIL-SWIGLU", 1, 1),)),
    "f32-301": Case(F_SHORT, 301, (("PART", 2, 0), ("PART", 2, 1), ("QKV", 3, 0))),
    "f32-403": Case(F_SHORT, 403, (("QKV", 2, 0), ("SWIGLU", 4, 0)), oracle=False),
    "f32-1001": Case(F_SHORT, 1001, (("PART", 3, 0), ("QKV", 4, 0), ("SWIGLU", 3, 0)), oracle=False),
    "f32-mha-101": Case(F_MHA, 101, (("TAIL-QKV", 1, 1),)),
    "f32-mha-249": Case(F_MHA, 249, (("TAIL-QKV", 2, 1),), oracle=False),
    "f32-mha-333": Case(F_MHA, 333, (("TAIL-QKV", 3, 1),), oracle=False),
    "f32-2k-131": Case(F_2K, 131, (("TAIL-SWIGLU", 3, 0),), oracle=False),
    "f32-2k-703": Case(F_2K, 703, (("TAIL-SWIGLU", 4, 1),), oracle=False),
    "f32-wide-901": Case(F_WIDE, 901, (("TAIL-QKV", 4, 1),), oracle=False),
    "f32-long-21": Case(F_LONG, 21, (("PART", 2, 1), ("QKV", 1, 1), ("SWIGLU", 1, 1))),
    "f32-long-61": Case(F_LONG, 61, (("PART", 2, 1), ("QKV", 1, 1), ("SWIGLU", 2, 1), ("TAIL-SWIGLU", 2, 0))),
    "f32-long-403": Case(F_LONG, 403, (("PART", 3, 0), ("PART", 3, 1), ("QKV", 2, 1), ("SWIGLU", 4, 0)), oracle=False),
    "f32-long-601": Case(F_LONG, 601, (("PART", 4, 0), ("QKV", 3, 1), ("SWIGLU", 2, 1), ("TAIL-QKV", 3, 0), ("TAIL-SWIGLU", 2, 1)),
                         oracle=False),
    "f32-long-901": Case(F_LONG, 901, (("PART", 3, 1), ("QKV", 4, 0), ("SWIGLU", 3, 1), ("TAIL-SWIGLU", 3, 1)), oracle=False),
    "bf16-ffn-777": Case(B_FFN, 777, (("SWIGLU", 4, 4, 8),)),
    "bf16-ffn-1950": Case(B_FFN, 1950, (("SWIGLU", 8, 4, 4),)),
    "bf16-ffn-2301": Case(B_FFN, 2301, (("SWIGLU", 4, 4, 4),), oracle=False, chunk=8192),
    "bf16-wide-1500": Case(B_WIDE, 1500, (("RESID", 4, 4, 4), ("STORE", 4, 4, 4))),
    "bf16-wide-2501": Case(B_WIDE, 2501, (("RESID", 8, 4, 4), ("STORE", 8, 4, 4)), oracle=False, chunk=8192),
    "bf16-odd-1500": Case(B_ODD, 1500, (("RESID", 4, 4, 8), ("STORE", 4, 4, 8)), oracle=False),
    "bf16-qkv-1901": Case(B_QKV2, 1901, (("QKV", 4, 4, 4),), oracle=False),
    "bf16-qkv-3100": Case(B_QKV, 3100, (("QKV", 4, 4, 8),), oracle=False, chunk=8192),
    "bf16-qkv-8100": Case(B_QKV, 8100, (("QKV", 8, 4, 4), ("SWIGLU", 4, 4, 8)), oracle=False, chunk=8192),
    "bf16-split-50": Case(B_SPLIT, 50, (("PART", 4, 2, 8), ("PART", 4, 3, 8))),
    "bf16-split-101": Case(B_SPLIT, 101, (("PART", 8, 2, 8), ("PART", 8, 3, 8))),
}


def rows_of(src, cfg, slots):
    """K and V rows of the target layer and of the draft head (behind all of the layer's GEMMs)."""
    return {(layer, which): np.stack([src.kv_row(layer, which, s) for s in slots]) for layer in (0, 1) for which in (0, 1)}


def compare(cfg, a, b):
    for key in a:
        if cfg.dtype == FP32:   # the bar of the parity tests, for values of order one
            assert np.max(np.abs(a[key] - b[key])) <= 1e-4 * max(1.0, float(np.std(a[key]))), key
        else:   # a flipped bf16 rounding is 2^-8 of an element
            assert np.max(np.abs(a[key] - b[key])) <= np.max(np.abs(a[key])) * 2 ** -7 + 1e-6, key
            assert np.mean(a[key] != b[key]) < (0.02 if key[0] == 0 else 0.3), key


@pytest.mark.parametrize("name", CASES)
def test_every_row_of_every_tile(name):
    c = CASES[name]
    cfg, tol = c.config, 1e-4 if c.cfg.dtype == FP32 else 2e-2
    if c.oracle:
        eng, orc, _ = make_pair(cfg, 101)
    else:
        eng, orc = Engine(cfg, to_device(synth.make_weights(cfg, 101))), None
    ids = synth.token_ids(c.n, cfg.vocab, 102)
    slots = list(range(c.n - 1))
    got = {}
    for mode in (Engine.PREFILL_BLOCKS, Engine.PREFILL_AUTO):
        eng.set_prefill_mode(mode, c.chunk)
        eng.prefill(ids)
        got[mode] = eng.logits(0), rows_of(eng, cfg, slots)
    (lb, rb), (la, ra) = got[Engine.PREFILL_BLOCKS], got[Engine.PREFILL_AUTO]
    assert np.max(np.abs(lb - la)) <= tol
    compare(cfg, rb, ra)
    if orc is not None:
        orc.prefill(ids)
        assert np.max(np.abs(orc.logits(0) - la)) <= tol
        compare(cfg, rows_of(orc, cfg, slots), ra)
    eng.close()
