"""What the workgroups of the bf16 prompt GEMMs read of a chunk's rows (host code over a recorded HIP runtime, no GPU): no row-block
behind the chunk's buffers, every row that there is, in the same number of loads a wave."""
import re

import pytest

from paper_2412_18910_amd.binding import AE_OK
from paper_2412_18910_amd.config import BF16, Config

from .fake_runtime import Ctx
from .test_gpu_prompt_plans import CASES, _cfg
from .test_gpu_prompt_tiles import CASES as TILES

SHAPES = [Config(1, 4096, 32, 32, 128, 11008, 512, dtype=BF16), Config(1, 5120, 40, 40, 128, 13824, 512, dtype=BF16),
          Config(1, 4096, 32, 8, 128, 14336, 512, dtype=BF16)]
LONG = [(cfg, n, 0) for cfg in SHAPES for n in (61, 100, 333, 1136, 2048, 2200, 4096)]
OTHERS = [(_cfg(*c[0]), c[1], 8192) for c in CASES if BF16 in c[0][4:] or len(c[0]) == 4] + \
    [(c.cfg, c.n, c.chunk) for c in TILES.values() if c.cfg.dtype == BF16]


def gemms(cfg, n, chunk):
    """(row-blocks of a tile, waves) of the GEMMs of a prompt of one chunk."""
    c = Ctx(cfg.with_(n_ctx_max=n + 16, k_max=5, ldlp_hidden=64))
    assert c.prefill_mode(0, chunk) == AE_OK
    c.lib.fake_clear()
    assert c.prefill(n) == AE_OK
    out = [(int(m[1]), int(m[2])) for name, *_ in c.launches()
           if (m := re.search(r"gemm_dense_kernelILi\dELb\dELi(\d)ELi\dELi(\d)E", name))]
    lib = c.lib
    c.close()
    return lib, out


@pytest.mark.parametrize("cfg,n,chunk", LONG + OTHERS, ids=lambda v: str(v.d_model) if isinstance(v, Config) else str(v))
def test_tiles_are_read_where_there_are_any(cfg, n, chunk):
    lib, launched = gemms(cfg, n, chunk)
    assert len(launched) == 6   # a plan that is launched for QKV, o, gate/up and down, and for the draft head's two
    RB = (n + 127) // 128 * 8
    for dm, nw in set(launched):
        loads = (2 * dm + nw - 1) // nw
        for rows in (n, n - 1):   # of the layer, of the draft head
            for rb0 in range(0, (rows + 15) // 16, dm):
                got = {}
                for w in range(nw):
                    for i in range(loads):
                        slot = lib.fake_dense_slot(w, i, nw, dm)
                        assert 0 <= slot < 2 * dm
                        got.setdefault(slot, set()).add(rb0 * 2 + lib.fake_dense_source(slot, rb0, RB))
                assert len(got) == 2 * dm and all(len(s) == 1 for s in got.values())
                assert max(max(s) for s in got.values()) < 2 * RB, (dm, rb0, RB)
                for slot, (tile,) in got.items():   # rows come from their own place
                    assert tile == rb0 * 2 + slot or rb0 * 2 + slot >= 2 * ((rows + 15) // 16)
