"""Performance cases of the AdaEAGLE engine: prompts, verification blocks and whole decode steps at
batch size 1, timed through the Engine's public calls, with a float64 re-expression of what each
returns.

A case is a dict of plain values:
  kind     "prompt" (Engine.prefill), "verify" (Engine.verify of a block) or "step" (Engine.step)
  shape    a preset of the package ("tiny", "7b", "13b", "8b-gqa") or "small", a grouped-query
           model of the size used by the parity tests
  dtype    "bf16" or "fp32": matrices and KV cache
  layers   decoder layers of the target (the widths are the shape's own, the depth is cut where the
           whole model would only repeat the same layers)
  context  tokens in the cache (prompt: tokens of the prompt)
  rows     verify: rows of the block; step: draft tokens (k), the block then has k + 1 rows
  t        temperature; 0 is greedy
  ddd      1: the log-probability exit rule of the draft head is on
"""
import math

import numpy as np
import torch

from paper_2412_18910_amd.binding import Engine
from paper_2412_18910_amd.config import BF16, FP32, PRESETS, Config

DEV = "cuda"
SMALL = Config(3, 256, 8, 2, 64, 512, 2048, dtype=BF16, k_max=6, ldlp_hidden=64, rope_base=500000.0, rms_eps=1e-5)


def _case(name, kind, shape, dtype, layers, context, rows, t=0.0, ddd=0):
    return {"name": name, "kind": kind, "shape": shape, "dtype": dtype, "layers": layers, "context": context,
            "rows": rows, "t": t, "ddd": ddd}


def listed():
    return [
        # the smallest model of the package: every kernel is tiny, launches and host work are the time
        _case("tiny_fp32_step", "step", "tiny", "fp32", 2, 64, 4),
        # plain autoregressive decoding, one row a pass: the baseline that every speculative run is held against
        _case("7b_verify_1", "verify", "7b", "bf16", 8, 1024, 1),
        # the widest block the 13B shape verifies (k_max 10), in the middle of a long conversation
        _case("13b_verify_11", "verify", "13b", "bf16", 8, 4096, 11),
        # grouped queries, a document of odd length in the cache, large vocabulary
        _case("8b_gqa_verify_9", "verify", "8b-gqa", "bf16", 8, 8001, 9),
        # the headline: one whole decode step of the full 7B model at 2048 tokens
        _case("7b_step", "step", "7b", "bf16", 32, 2048, 4),
        # lossless sampling over 128256 tokens; the temperature makes the random head's drafts acceptable
        _case("8b_gqa_step_sampled", "step", "8b-gqa", "bf16", 4, 1999, 4, t=26.0),
        # the exit rule of the draft head, early in a chat: short drafts, block padded to k_max + 1 rows
        _case("7b_step_ddd", "step", "7b", "bf16", 4, 517, 2, ddd=1),
        # a long prompt through the full 7B model
        _case("7b_prompt_2048", "prompt", "7b", "bf16", 32, 2048, 0),
        # a short chat prompt, no multiple of any tile
        _case("7b_prompt_100", "prompt", "7b", "bf16", 8, 100, 0),
        # a document: several chunks, attention over thousands of keys, a ragged end
        _case("8b_gqa_prompt_7777", "prompt", "8b-gqa", "bf16", 4, 7777, 0),
        # float32 weights and cache, the precision the method was published with: decode and prompt
        _case("7b_fp32_step", "step", "7b", "fp32", 4, 300, 4),
        _case("7b_fp32_prompt_333", "prompt", "7b", "fp32", 4, 333, 0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("prompt", "verify", "verify", "step", "step"))
    shape, dtype, deepest, longest = rng.choice((
        ("tiny", "fp32", 3, 300), ("small", "bf16", 4, 600), ("7b", "bf16", 8, 4096), ("7b", "bf16", 8, 4096),
        ("13b", "bf16", 8, 4096), ("8b-gqa", "bf16", 8, 8192), ("8b-gqa", "bf16", 8, 8192), ("7b", "fp32", 4, 600)))
    k_max = _base(shape).k_max
    c = {"kind": kind, "shape": shape, "dtype": dtype, "layers": rng.randint(1, deepest),
         "context": _log_int(rng, 3, longest), "rows": 0, "t": 0.0, "ddd": 0}
    if kind == "verify":
        c["rows"] = rng.randint(1, k_max + 1)
    elif kind == "step":
        c["rows"] = rng.randint(1, k_max)
        c["ddd"] = int(rng.random() < 0.25)
        c["t"] = 26.0 if not c["ddd"] and rng.random() < 0.35 else 0.0
    return c


# ---------------------------------------------------------------------------- inputs
def _base(shape):
    return SMALL if shape == "small" else PRESETS[shape]


def _config(case):
    base = _base(case["shape"])
    return base.with_(n_layers=case["layers"], dtype=BF16 if case["dtype"] == "bf16" else FP32,
                      n_ctx_max=case["context"] + base.k_max + 2, temperature=case["t"], ddd_enabled=case["ddd"])


def _weights(cfg, seed):
    """Random-init weights: matrices N(0, 0.02^2), gains around one, small biases."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    mdt = torch.bfloat16 if cfg.dtype == BF16 else torch.float32

    def mat(*shape):
        return torch.empty(*shape, dtype=mdt, device=DEV).normal_(0.0, 0.02, generator=g)

    def vec(n, mean, std):
        return torch.empty(n, dtype=torch.float32, device=DEV).normal_(mean, std, generator=g)

    d, f, v, h = cfg.d_model, cfg.d_ffn, cfg.vocab, cfg.ldlp_hidden
    dq, dkv = cfg.n_heads * cfg.head_dim, cfg.d_kv

    def layer():
        return {"attn_norm": vec(d, 1.0, 0.1), "wq": mat(dq, d), "wk": mat(dkv, d), "wv": mat(dkv, d), "wo": mat(d, dq),
                "ffn_norm": vec(d, 1.0, 0.1), "w_gate": mat(f, d), "w_up": mat(f, d), "w_down": mat(d, f)}

    w = {"tok_emb": mat(v, d), "lm_head": mat(v, d), "final_norm": vec(d, 1.0, 0.1),
         "layers": [layer() for _ in range(cfg.n_layers)], "draft_layer": layer(), "draft_fc_w": mat(d, 2 * d),
         "draft_fc_b": vec(d, 0.0, 0.02), "ldlp_w_in": mat(h, 2 * d), "ldlp_b_in": vec(h, 0.0, 0.02),
         "ldlp_w_res": None, "ldlp_b_res": None,
         "ldlp_w_out": vec(h, 0.0, cfg.k_max / 4.0 / (math.sqrt(h * d) * 0.012)), "ldlp_b_out": vec(1, 4.0, 0.1)}
    return w


def _inputs(case, cfg, seed):
    """Prompt ids, the token pending behind them, the tokens of the block / draft, the uniforms of a sampled step."""
    r = np.random.Generator(np.random.Philox(seed))
    ids = r.integers(0, cfg.vocab, case["context"], dtype=np.int32)
    pending = int(r.integers(0, cfg.vocab))
    toks = r.integers(0, cfg.vocab, cfg.k_max + 1, dtype=np.int32)
    return ids, pending, toks, r.random(cfg.k_max), r.random(cfg.k_max + 1)


def prepare(case, seed):
    """An engine over random weights; for verify and step its caches hold the context.

    The tokens that the draft and the block run over are fixed by the seed (a step's through its override
    table), so that near ties of random logits cannot send two correct implementations to different inputs."""
    cfg = _config(case)
    eng = Engine(cfg, _weights(cfg, seed))
    ids, pending, toks, u_draft, u_accept = _inputs(case, cfg, seed)
    st = {"case": case, "cfg": cfg, "eng": eng, "ids": ids}
    if case["kind"] != "prompt":
        eng.prefill(ids)
        st["pending"], st["last"] = pending, int(ids[-1])
        st["feat"] = eng.feature((len(ids) - 1) % 16)
        if case["kind"] == "verify":
            st["block"] = np.concatenate([[pending], toks]).astype(np.int32)[:case["rows"]]
        else:
            st["override"] = toks[:cfg.k_max]
            st["u_draft"], st["u_accept"] = u_draft, u_accept
    return st


def run(state):
    eng, case = state["eng"], state["case"]
    if case["kind"] == "prompt":
        eng.prefill(state["ids"])
        return {"logits": eng.logits(0), "feature": eng.feature((len(state["ids"]) - 1) % 16), "y": eng.ldlp()[1]}
    if case["kind"] == "verify":
        eng.verify(state["block"])
        return {"logits": [eng.logits(i) for i in range(case["rows"])]}
    # the sequence is put back to where the step starts, then one iteration of the decode loop
    k = case["rows"]
    eng.set_state(len(state["ids"]), state["last"], state["pending"], state["feat"])
    if case["t"] > 0:
        k, acc, toks = eng.step(k, state["override"][:k], state["u_draft"][:k], state["u_accept"][:k + 1])
    else:
        k, acc, toks = eng.step(k, state["override"])
    out = {"draft": [eng.draft_logits(i) for i in range(k)], "logits": [eng.logits(i) for i in range(k + 1)],
           "k": int(k), "accepted": int(acc), "y": eng.ldlp()[1]}
    if case["t"] == 0:   # the logit of the token that the step settled on: near ties give the same value
        out["picked"] = float(out["logits"][acc][toks[-1]])
    return out


# ---------------------------------------------------------------------------- what a pass cannot do without
def work(case):
    cfg = _config(case)
    d, f, v, n = cfg.d_model, cfg.d_ffn, cfg.vocab, case["context"]
    dq, dkv, size = cfg.n_heads * cfg.head_dim, cfg.d_kv, 2 if cfg.dtype == BF16 else 4
    layer = 2 * d * dq + 2 * d * dkv + 3 * d * f
    ldlp = cfg.ldlp_hidden * 2 * d
    if case["kind"] == "prompt":
        draft = 2 * d * d + d * 2 * dkv   # of the draft head only the prompt's keys and values are needed
        flops = 2 * n * (cfg.n_layers * layer + draft) + 4 * cfg.n_layers * dq * n * (n + 1) // 2 + 2 * v * d
        rows_io = n * d + (cfg.n_layers + 1) * n * 2 * dkv
        return {"bytes": size * (cfg.n_layers * layer + draft + v * d + ldlp + rows_io) + 4 * v, "flops": flops}
    rows = case["rows"] if case["kind"] == "verify" else case["rows"] + 1
    # every weight once, the cached keys and values once, the logits once
    data = size * (cfg.n_layers * (layer + 2 * (n + rows) * dkv) + v * d) + 4 * rows * v
    flops = 2 * rows * (cfg.n_layers * layer + v * d) + 4 * cfg.n_layers * dq * n * rows
    if case["kind"] == "step":   # a chain: each draft token waits for the one before it and reads the head again
        k = case["rows"]
        data += k * (size * (2 * d * d + layer + v * d + 2 * n * dkv) + 4 * v) + size * ldlp
        flops += k * (2 * (2 * d * d + layer + v * d) + 4 * dq * n)
    return {"bytes": data, "flops": flops}


def tolerance(case):
    # About four times the largest error against float64 over listed and drawn cases: 4e-6 in float32; in bf16 2e-3 at
    # most depths, 4.6e-3 for long draft chains at the 13B widths (a bf16 cache adds roundings that flip, each 2^-9 of
    # one element, and every layer carries them on).  Of ~1e5 values the farthest is about five deviations off.
    if case["dtype"] == "fp32":
        return {"rel": 2e-5, "max": 2e-4}
    return {"rel": 1e-2, "max": 1e-1}


# ---------------------------------------------------------------------------- float64
class _Model64:
    """The method's forwards in float64; with a bf16 cache keys and values are rounded to bf16 where they are cached,
    as the engine's interface defines."""

    def __init__(self, cfg, w):
        self.cfg, self.w = cfg, w
        self.cache = [[None, None] for _ in range(cfg.n_layers + 1)]

    def cached(self, x):
        return x.to(torch.bfloat16).double() if self.cfg.dtype == BF16 else x

    def norm(self, x, gain):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + self.cfg.rms_eps) * gain.double()

    def emb(self, ids):
        return self.w["tok_emb"][torch.as_tensor(np.asarray(ids), dtype=torch.long, device=DEV)].double()

    def rope(self, x, pos0):
        hd = self.cfg.head_dim
        inv = self.cfg.rope_base ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64, device=DEV) / hd)
        ang = torch.arange(pos0, pos0 + x.shape[0], dtype=torch.float64, device=DEV)[:, None] * inv
        c, s = ang.cos()[:, None, :], ang.sin()[:, None, :]
        a, b = x[..., :hd // 2], x[..., hd // 2:]
        return torch.cat([a * c - b * s, b * c + a * s], -1)

    def layer(self, li, lw, x, pos0, attend=True):
        cfg, r = self.cfg, x.shape[0]
        h, hkv, hd = cfg.n_heads, cfg.n_kv_heads, cfg.head_dim
        y = self.norm(x, lw["attn_norm"])
        k = self.cached(self.rope((y @ lw["wk"].double().T).view(r, hkv, hd), pos0))
        v = self.cached((y @ lw["wv"].double().T).view(r, hkv, hd))
        ck, cv = self.cache[li]
        k = k if ck is None else torch.cat([ck[:pos0], k])
        v = v if cv is None else torch.cat([cv[:pos0], v])
        self.cache[li] = [k, v]
        if not attend:
            return None
        q = self.rope((y @ lw["wq"].double().T).view(r, h, hd), pos0)
        hidden = torch.arange(k.shape[0], device=DEV)[None, :] > torch.arange(pos0, pos0 + r, device=DEV)[:, None]
        att = torch.empty(r, h, hd, dtype=torch.float64, device=DEV)
        for i in range(h):
            s = (q[:, i] @ k[:, i // (h // hkv)].T / math.sqrt(hd)).masked_fill(hidden, -math.inf)
            att[:, i] = torch.softmax(s, -1) @ v[:, i // (h // hkv)]
        x = x + att.reshape(r, h * hd) @ lw["wo"].double().T
        y = self.norm(x, lw["ffn_norm"])
        g, u = y @ lw["w_gate"].double().T, y @ lw["w_up"].double().T
        return x + (torch.nn.functional.silu(g) * u) @ lw["w_down"].double().T

    def target(self, ids, pos0):
        """Feature rows (behind the final norm) of the tokens at slots pos0.."""
        x = self.emb(ids)
        for li in range(self.cfg.n_layers):
            x = self.layer(li, self.w["layers"][li], x, pos0)
        return self.norm(x, self.w["final_norm"])

    def head(self, x):
        return x @ self.w["lm_head"].double().T

    def draft(self, feat, next_ids, slot0, attend=True):
        x = torch.cat([feat, self.emb(next_ids)], -1) @ self.w["draft_fc_w"].double().T + self.w["draft_fc_b"].double()
        return self.layer(self.cfg.n_layers, self.w["draft_layer"], x, slot0, attend)

    def ldlp(self, tok, f):
        z = self.w["ldlp_w_in"].double() @ torch.cat([self.emb([tok])[0], f]) + self.w["ldlp_b_in"].double()
        return float(self.w["ldlp_w_out"].double() @ torch.nn.functional.silu(z) + self.w["ldlp_b_out"].double()[0])


def exact(case, seed):
    cfg = _config(case)
    m = _Model64(cfg, _weights(cfg, seed))
    ids, pending, toks, _, u_accept = _inputs(case, cfg, seed)
    n = len(ids)
    feats = m.target(ids, 0)
    if case["kind"] == "prompt":
        return {"logits": m.head(feats[-1]).cpu(), "feature": feats[-1].cpu(), "y": m.ldlp(ids[-1], feats[-1])}
    block = np.concatenate([[pending], toks])
    if case["kind"] == "verify":
        out = m.head(m.target(block[:case["rows"]], n))
        return {"logits": list(out.cpu())}
    k = case["rows"]
    if n > 1:
        m.draft(feats[:-1], ids[1:], 0, attend=False)
    draft, h = [], feats[-1:]
    for i in range(k):
        h = m.draft(h, [block[i]], n - 1 + i)
        draft.append(m.head(h[0]))
    f = m.target(block[:k + 1], n)
    logits = m.head(f)
    acc = 0
    if case["t"] > 0:
        for acc in range(k + 1):
            if acc == k:
                break
            p = torch.softmax(logits[acc] / case["t"], -1)[block[acc + 1]]
            q = torch.softmax(draft[acc] / case["t"], -1)[block[acc + 1]]
            if not u_accept[acc] < min(1.0, float(p / q)):
                break
    else:
        while acc < k and int(block[acc + 1]) == int(logits[acc].argmax()):
            acc += 1
    out = {"draft": [x.cpu() for x in draft], "logits": list(logits.cpu()), "k": k, "accepted": acc,
           "y": m.ldlp(block[acc], f[acc])}
    if case["t"] == 0:
        out["picked"] = float(logits[acc].max())
    return out
