"""The library's host code over tests/fake_hip.cpp: no GPU, kernels recorded instead of run."""
import ctypes as C
import os
import subprocess

import numpy as np

from paper_2412_18910_amd import binding, build
from paper_2412_18910_amd.binding import AeConfig, AeLayerW, AeStepIO, AeWeights

HERE = os.path.dirname(os.path.abspath(__file__))
_lib = None


def load():
    global _lib
    if _lib is None:
        objs = [os.path.join(build.OBJ_DIR, os.path.basename(s)[:-4] + ".o") for s in build.sources()]
        if build.is_stale() or not all(map(os.path.exists, objs)):
            build.build()
        out = os.path.join(build.OBJ_DIR, "fake", f"libadaeagle_fake_{os.getpid()}.so")
        os.makedirs(os.path.dirname(out), exist_ok=True)
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__",
                               "-I/opt/rocm/include", "-I", os.path.join(build.ROOT, "include"), "-I", os.path.join(build.HERE, "csrc"),
                               "-Wno-unused-result", "-o", out, os.path.join(HERE, "fake_hip.cpp")] + objs)
        saved, binding._lib = binding._lib, None
        try:
            _lib = binding.load_library(out)
        finally:
            binding._lib = saved
            os.remove(out)
        _lib.fake_name.restype = C.c_char_p
        _lib.fake_live_bytes.restype = C.c_size_t
        _lib.fake_fail_alloc.argtypes = [C.c_size_t]
        _lib.fake_room.argtypes = [C.c_size_t]
        _lib.fake_fail_launch.argtypes = [C.c_long]
    return _lib


class Ctx:
    """A context of the C ABI whose weights nobody reads."""

    def __init__(self, cfg, bias=True):
        self.lib, self.cfg = load(), cfg
        dummy = C.c_void_p(4096)
        layer = AeLayerW(**{n: dummy for n, _ in AeLayerW._fields_})
        self._layers = (AeLayerW * cfg.n_layers)(*[layer] * cfg.n_layers)
        w = AeWeights(**{n: dummy for n, _ in AeWeights._fields_ if n not in ("layers", "draft_layer")})
        w.layers, w.draft_layer = C.cast(self._layers, C.POINTER(AeLayerW)), layer
        if not bias:
            w.draft_fc_b = None
        self.h = C.c_void_p()
        rc = self.lib.ae_init(C.byref(AeConfig(**cfg.dict())), C.byref(w), None, C.byref(self.h))
        assert rc == 0, self.lib.ae_last_error(None)

    def close(self):
        self.lib.ae_free(self.h)

    def prefill(self, n):
        ids = np.zeros(n, np.int32)
        return self.lib.ae_prefill(self.h, ids.ctypes.data_as(C.POINTER(C.c_int32)), n)

    def prefill_mode(self, mode, chunk=0):
        return self.lib.ae_set_prefill_mode(self.h, mode, chunk)

    def set_state(self, n):
        feat = np.zeros(self.cfg.d_model, np.float32)
        return self.lib.ae_set_state(self.h, n, 0, 0, feat.ctypes.data_as(C.POINTER(C.c_float)))

    def verify(self, rows, implicit=False):
        ids = np.zeros(rows, np.int32)
        return self.lib.ae_verify(self.h, None if implicit else ids.ctypes.data_as(C.POINTER(C.c_int32)), rows)

    def draft(self, k):
        return self.lib.ae_draft(self.h, k, None, None, None)

    def accept(self):
        n, b = C.c_int(), C.c_int32()
        return self.lib.ae_accept(self.h, None, C.byref(n), C.byref(b))

    def step(self, k):
        io = AeStepIO()
        io.k_force = k
        return self.lib.ae_step(self.h, C.byref(io)), io

    def _get(self, fn, n, *args):
        out = np.zeros(n, np.float32)
        return fn(self.h, *args, out.ctypes.data_as(C.POINTER(C.c_float)))

    def logits(self, row=0):
        return self._get(self.lib.ae_get_logits, self.cfg.vocab, row)

    def feature(self, row=0):
        return self._get(self.lib.ae_get_feature, self.cfg.d_model, row)

    def kv_row(self):
        return self._get(self.lib.ae_get_kv_row, self.cfg.d_kv, 0, 0, 0)

    def launches(self):
        """(kernel name, grid x, grid y, threads) since the last clear."""
        out = []
        for i in range(self.lib.fake_launches()):
            g = [C.c_uint() for _ in range(3)]
            self.lib.fake_grid(i, *[C.byref(x) for x in g])
            out.append((self.lib.fake_name(i).decode(),) + tuple(x.value for x in g))
        return out

    def count(self, fn):
        """Launches of one call, which has to succeed."""
        self.lib.fake_clear()
        assert fn() == 0
        return self.lib.fake_launches()
