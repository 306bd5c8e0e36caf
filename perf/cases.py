"""The work that users of the routed mixture-of-head attention library have it
do: prompts (prefill), training steps, the layer with its routed projections,
decode steps, and a prompt followed by generation.

Every case goes through ``paper_2609_38832_amd._lib`` the way a model's code
does: workspaces and outputs are allocated once and passed in, routing results
feed the attention, caches are updated in place.  Queries, keys and values are
N(0, 1) (what a projection of normalised activations gives), router logits
N(0, 1), with a Zipf-like per-head offset where routing is skewed.

Case fields (plain values; a kind reads those that it needs):
  kind     "prefill" | "train" | "layer" | "decode" | "serve"
  dtype    "bf16" | "f32"
  B, T     sequences, tokens of each (decode: T unused)
  H, K, d  routed heads (key/value groups when g > 1), selected ones, width
  g        query heads per key/value group
  zipf     logits += zipf * ln(1 / (h + 1))
  Hs, win  always-active shared heads and their window (0: the whole prefix)
  dm       model width of the projections
  packed   train: gradients of the routed pairs (else dense [B, H, T, d])
  biased   train: loss-free balancing routing (a fixed selection bias)
  prior    decode: tokens that each sequence has seen
  steps    decode/serve: generated tokens per pass
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2609_38832_amd import _lib as L

DEV = "cuda:0"
BASE = {"dtype": "bf16", "g": 1, "zipf": 0.0, "Hs": 0, "win": 0, "dm": 0, "packed": True,
        "biased": False, "prior": 0, "steps": 0, "rope_base": 1e4}


def _case(kind, name=None, **kw):
    c = dict(BASE, kind=kind, **kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # a short chat prompt, one sequence, the pretraining head layout
        # (32 heads, 8 active, width 64): launches and latency count
        _case("prefill", "prefill_short", B=1, T=300, H=32, K=8, d=64),
        # the pretraining batch: 4 sequences of 4096 tokens, balanced routing
        _case("prefill", "prefill_balanced", B=4, T=4096, H=32, K=8, d=64),
        # long context with skewed routing and ragged lengths, width 128
        _case("prefill", "prefill_skewed", B=2, T=15997, H=32, K=4, d=128, zipf=1.5),
        # long context with 64 query heads in key/value groups of 4 and two
        # shared heads over a sliding window added to the same output
        _case("prefill", "prefill_groups_shared", B=1, T=32768, H=16, K=2, d=128, g=4, Hs=2,
              win=1024, rope_base=5e5),
        # the layer with its Q/K/V and output projections at the pretraining
        # width (d_model 2048)
        _case("layer", "layer_dm2048", B=4, T=4096, H=32, K=8, d=64, dm=2048),
        # the layer at d_model 4096, heads of width 128, an odd token count
        _case("layer", "layer_dm4096", B=2, T=3001, H=32, K=8, d=128, dm=4096),
        # a pretraining step of the attention: route, forward that keeps its
        # state, gradients of the routed pairs, router gradient
        _case("train", "train_balanced", B=4, T=4096, H=32, K=8, d=64),
        # long-context fine-tuning with loss-free balancing, skewed, dense
        # gradients
        _case("train", "train_skewed", B=1, T=12289, H=32, K=4, d=128, zipf=1.5, packed=False,
              biased=True),
        # a float32 training step (numerics work, small models)
        _case("train", "train_f32", B=2, T=1000, H=16, K=4, d=64, dtype="f32", packed=False),
        # generation for one user after about a thousand tokens
        _case("decode", "decode_single", B=1, T=1, H=32, K=8, d=64, prior=1200, steps=8),
        # a serving batch deep into long contexts, 64 heads of width 128
        _case("decode", "decode_batch", B=64, T=1, H=64, K=8, d=128, prior=32768, steps=2,
              rope_base=5e5),
        # a request batch: prompt, hand-off to the caches, generation, with
        # key/value groups and windowed shared heads
        _case("serve", "serve_groups_shared", B=8, T=2043, H=16, K=4, d=128, g=4, Hs=2, win=512,
              steps=8),
    ]


# ---------------------------------------------------------------------------
# draws

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _most(kind):
    """The largest listed case's time estimate, of a kind."""
    return max(_cost(c) for c in listed() if c["kind"] == kind)


def _cost(c):
    """Rough seconds at the card's nominal rates (draws stay under the listed
    cases of their kind)."""
    w = work(c)
    return max(w["bytes"] / 5e12, w["flops"] / (6e14 if c["dtype"] == "bf16" else 2e13))


def _draw_once(rng):
    kind = rng.choice(["prefill", "prefill", "prefill", "train", "train", "layer", "decode",
                       "decode", "serve"])
    d = rng.choice([64, 128])
    c = _case(kind, d=d, rope_base=rng.choice([1e4, 5e5]), B=rng.choice([1, 1, 2, 3, 4, 8]), T=1,
              zipf=rng.choice([0.0, 0.0, 1.5]))
    c["H"] = rng.choice([8, 16, 32, 64])
    c["K"] = rng.choice([k for k in (1, 2, 4, 8, 12) if 2 * k <= c["H"]])
    if kind in ("prefill", "decode", "serve"):
        c["g"] = rng.choice([1, 1, 1, 2, 4])
    if kind == "prefill":
        c["T"] = _log_int(rng, 100, 32768)
        if rng.random() < 0.2:
            c["dtype"], c["g"], c["d"] = "f32", 1, rng.choice([32, 64, 128])
            c["T"] = _log_int(rng, 100, 2048)
        elif rng.random() < 0.3:
            c["Hs"], c["win"] = rng.choice([1, 2]), rng.choice([0, 128, 500, 2048])
            c["T"] = min(c["T"], 16384)
    elif kind == "train":
        c["T"] = _log_int(rng, 100, 16384)
        c["packed"], c["biased"] = rng.random() < 0.6, rng.random() < 0.4
        if rng.random() < 0.25:
            c["dtype"], c["d"] = "f32", rng.choice([32, 64, 128])
            c["T"] = _log_int(rng, 100, 1000)
    elif kind == "layer":
        c["T"], c["dm"] = _log_int(rng, 60, 4096), rng.choice([512, 1024, 1536, 2048, 4096])
    elif kind == "decode":
        c["B"], c["prior"] = _log_int(rng, 1, 64), _log_int(rng, 100, 131072)
        c["steps"], c["g"] = rng.choice([1, 2, 4]), rng.choice([c["g"], c["g"], 8])
        if rng.random() < 0.3:
            c["Hs"], c["win"] = rng.choice([1, 2]), rng.choice([128, 1000])
        c["zipf"] = 0.0
    else:
        c["T"], c["steps"] = _log_int(rng, 50, 4096), rng.choice([2, 4, 8])
        if rng.random() < 0.5:
            c["Hs"], c["win"] = rng.choice([1, 2]), rng.choice([128, 500])
    if c["g"] > 1:  # H and K count the groups
        c["H"] = max(4, c["H"] // c["g"])
        c["K"] = min(c["K"], c["H"] // 2)
    return c


def draw(rng):
    while True:
        c = _draw_once(rng)
        if _cost(c) > _most(c["kind"]):
            continue
        if c["kind"] == "decode" and _cache_bytes(c) > 13e9:
            continue
        # dense q, k, v (and gradients) of a state stay a few GB
        if c["kind"] != "decode" and c["B"] * c["H"] * c["g"] * c["T"] * c["d"] > 6e8:
            continue
        return c


# ---------------------------------------------------------------------------
# sizes

def _loads(c):
    """Expected rows of each head (n / T) of one sequence, from a fixed
    sample of the router logits' distribution."""
    if not c["zipf"]:
        return np.full(c["H"], c["K"] / c["H"])
    z = np.random.default_rng(1).standard_normal((4096, c["H"]))
    z += c["zipf"] * np.log(1.0 / (np.arange(c["H"]) + 1.0))
    if c["biased"]:
        z = np.exp(z - z.max(1, keepdims=True))
        z = z / z.sum(1, keepdims=True) + _bias_np(c["H"])
    top = np.argpartition(-z, c["K"] - 1, axis=1)[:, :c["K"]]
    return np.bincount(top.ravel(), minlength=c["H"]) / 4096.0


def _bias_np(H):
    """A balancing bias part of the way to balance: later heads are favoured."""
    return 0.02 * np.arange(H) / H


def _cap(c):
    if c["kind"] == "serve":
        return c["T"] + c["steps"]
    mean = c["prior"] * c["K"] / c["H"]
    return (int(mean * 1.25) + c["steps"] + 255) // 256 * 256


def _cache_bytes(c):
    return 4 * c["B"] * c["H"] * _cap(c) * c["d"]


def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    B, T, H, K, d, g = (c[n] for n in ("B", "T", "H", "K", "d", "g"))
    rows = B * T * K
    n = T * _loads(c)
    pairs = g * B * float((n * (n + 1) / 2).sum())
    logits = 4 * B * T * H
    qkv = rows * d * e * (g + 2)
    if c["Hs"]:
        w = min(c["win"] or T, T)
        spairs = B * c["Hs"] * (w * (w + 1) / 2 + (T - w) * w)
        sbytes = 3 * B * c["Hs"] * T * d * e
    else:
        spairs = sbytes = 0
    if c["kind"] == "prefill":
        return {"bytes": logits + qkv + 20 * rows + B * T * d * e + sbytes,
                "flops": 4.0 * d * (pairs + spairs)}
    if c["kind"] == "train":
        grads = 4 * d * 3 * (rows if c["packed"] else B * T * H)
        return {"bytes": 2 * logits + 2 * qkv + 24 * rows + grads + B * T * d * (e + 4),
                "flops": 14.0 * d * pairs}
    if c["kind"] == "layer":
        dm = c["dm"]
        return {"bytes": logits + 20 * rows + 2 * B * T * dm * 2 + 4 * H * d * dm * 2,
                "flops": 8.0 * rows * d * dm + 4.0 * d * pairs}
    # decode steps: the selected heads' cached rows
    if c["kind"] == "decode":
        m, prompt_b, prompt_f = c["prior"] * K / H, 0, 0
        srows = min(c["win"] or c["prior"], c["prior"])
    else:
        m = float((n * n).sum() / max(n.sum(), 1))
        srows = min(c["win"] or T, T)
        prompt_b = logits + qkv + 20 * rows + B * T * d * e + sbytes + 2 * rows * d * e
        prompt_b += 2 * B * c["Hs"] * srows * d * e
        prompt_f = 4.0 * d * (pairs + spairs)
    step_b = 2 * d * e * (B * K * (m + 2) + B * c["Hs"] * (srows + 2))
    step_f = 4.0 * d * B * (K * g * m + c["Hs"] * srows)
    return {"bytes": prompt_b + c["steps"] * step_b, "flops": prompt_f + c["steps"] * step_f}


def tolerance(case):
    # About four times the largest relative error of an output against the
    # 64-bit reference, measured over the listed cases and draws.
    # float32 (5e-7 seen): float32 sums.  bf16: rotated queries and keys,
    # probabilities and outputs rounded to bf16 (2^-9 each); the layer rounds
    # q, k, v and the gated head rows too; a decode step rounds its output and
    # the appended rows (with groups of 4 and more, queries and probabilities).
    if case["dtype"] == "f32":
        return {"rel": 2e-6}
    return {"rel": {"prefill": 1.3e-2, "serve": 1.3e-2, "layer": 1.8e-2, "train": 1.5e-2,
                    "decode": 1e-2}[case["kind"]]}


# ---------------------------------------------------------------------------
# inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _randn(gen, *shape, dtype=torch.float32, scale=1.0):
    x = torch.randn(*shape, generator=gen, device=DEV, dtype=dtype)
    return x if scale == 1.0 else x.mul_(scale)


def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _logits(c, gen, *lead):
    x = _randn(gen, *lead, c["H"])
    if c["zipf"]:
        off = c["zipf"] * np.log(1.0 / (np.arange(c["H"]) + 1.0))
        x += torch.tensor(off, dtype=torch.float32, device=DEV)
    return x


def _routing_out(B, T, H, K):
    i32 = dict(dtype=torch.int32, device=DEV)
    return {"topk_idx": torch.empty(B, T, K, **i32),
            "gates": torch.empty(B, T, K, dtype=torch.float32, device=DEV),
            "head_len": torch.empty(B, H, **i32), "seg_offsets": torch.empty(B * H + 1, **i32),
            "perm_token": torch.empty(B * T * K, **i32), "slot_pos": torch.empty(B, T, K, **i32)}


def _inputs(c, gen):
    """The tensors a program holds before the call (and that exact() reads)."""
    B, T, H, K, d, g, dt = (*(c[n] for n in ("B", "T", "H", "K", "d", "g")), _dtype(c))
    s = {}
    if c["kind"] == "layer":
        dm = c["dm"]
        s["logits"] = _logits(c, gen, B, T)
        s["x"] = _randn(gen, B, T, dm, dtype=dt)
        s["w_qkv"] = _randn(gen, H, 3, d, dm, dtype=dt, scale=dm ** -0.5)
        s["w_o"] = _randn(gen, H, dm, d, dtype=dt, scale=(K * d) ** -0.5)
        return s
    if c["kind"] != "decode":
        s["logits"] = _logits(c, gen, B, T)
        s["q"] = _randn(gen, B, H * g, T, d, dtype=dt)
        s["k"] = _randn(gen, B, H, T, d, dtype=dt)
        s["v"] = _randn(gen, B, H, T, d, dtype=dt)
        if c["Hs"]:
            s["qs"], s["ks"], s["vs"] = (_randn(gen, B, c["Hs"], T, d, dtype=dt) for _ in range(3))
    if c["kind"] == "train":
        s["dout"] = _randn(gen, B, T, d)
        if c["biased"]:
            s["bias"] = torch.tensor(_bias_np(H), dtype=torch.float32, device=DEV)
    if c["steps"]:
        S, cap = c["steps"], _cap(c)
        s["step_logits"] = _logits(c, gen, S, B)
        s["step_q"] = _randn(gen, S, B, H * g, d, dtype=dt)
        s["step_k"], s["step_v"] = (_randn(gen, S, B, H, d, dtype=dt) for _ in range(2))
        if c["Hs"]:
            s["step_qs"], s["step_ks"], s["step_vs"] = (
                _randn(gen, S, B, c["Hs"], d, dtype=dt) for _ in range(3))
        if c["kind"] == "decode":
            mean = c["prior"] * K / H
            n = torch.round(mean * (1 + 0.05 * _randn(gen, B, H))).clamp_(0, cap - S)
            s["len0"] = n.to(torch.int32)
            s["k_cache"], s["v_cache"] = (_randn(gen, B, H, cap, d, dtype=dt) for _ in range(2))
            if c["Hs"]:
                s["slen0"] = torch.full((B,), c["prior"], dtype=torch.int32, device=DEV)
                s["ks_cache"], s["vs_cache"] = (
                    _randn(gen, B, c["Hs"], c["win"], d, dtype=dt) for _ in range(2))
        else:
            s["k_cache"], s["v_cache"] = (torch.zeros(B, H, cap, d, dtype=dt, device=DEV)
                                          for _ in range(2))
            if c["Hs"]:
                s["ks_cache"], s["vs_cache"] = (
                    torch.zeros(B, c["Hs"], c["win"], d, dtype=dt, device=DEV) for _ in range(2))
    return s


def prepare(case, seed):
    c = case
    B, T, H, K, d, g, dt = (*(c[n] for n in ("B", "T", "H", "K", "d", "g")), _dtype(c))
    s = _inputs(c, _gen(seed))
    s["c"] = c
    f32 = dict(dtype=torch.float32, device=DEV)
    if c["kind"] != "decode":
        s["r"] = _routing_out(B, T, H, K)
        s["rws"] = L.workspace(L.route_workspace_size(B, T, H, K), DEV)
        s["out"] = torch.empty(B, T, d, dtype=dt, device=DEV)
    code = L.dtype_code(dt)
    lib = L.lib()
    if c["kind"] in ("prefill", "serve"):
        if g > 1:
            n = lib.namoh_attn_fwd_grouped_workspace_size(B, T, H, K, g, d, code)
        else:
            n = L.attn_workspace_size(B, T, H, K, d, code)
        s["aws"] = L.workspace(int(n), DEV)
        if c["Hs"]:
            s["sws"] = L.workspace(int(lib.namoh_shared_attn_workspace_size(B, T, c["Hs"], d)), DEV)
    elif c["kind"] == "layer":
        dm = c["dm"]
        s["qkv"] = {n: torch.empty(B, H, T, d, dtype=dt, device=DEV) for n in ("q", "k", "v")}
        s["aws"] = L.workspace(L.attn_workspace_size(B, T, H, K, d, code), DEV)
        s["head_out"] = torch.empty(B * T * K, d, **f32)
        s["ows"] = L.workspace(L.out_proj_workspace_size(B, T, H, K, d, dm), DEV)
        s["out"] = torch.empty(B, T, dm, dtype=dt, device=DEV)
    elif c["kind"] == "train":
        s["bws"] = L.workspace(int(lib.namoh_attn_bwd_workspace_size(B, T, H, K, d)), DEV)
        if dt == torch.float32:
            s["aws"] = L.workspace(L.attn_workspace_size(B, T, H, K, d, code), DEV)
        shape = (B * T * K, d) if c["packed"] else (B, H, T, d)
        s["grads"] = {n: torch.empty(*shape, **f32) for n in ("dq", "dk", "dv")}
        s["grads"]["dgates"] = torch.empty(B, T, K, **f32)
    if c["steps"]:
        cap = _cap(c)
        s["len"] = torch.zeros(B, H, dtype=torch.int32, device=DEV)
        if g > 1:
            n = lib.namoh_decode_grouped_workspace_size(B, H, K, g, d, cap)
        else:
            n = L.decode_workspace_size(B, H, K, d, cap)
        s["dws"] = L.workspace(int(n), DEV)
        if c["Hs"]:
            s["slen"] = torch.zeros(B, dtype=torch.int32, device=DEV)
            s["dsws"] = L.workspace(
                int(lib.namoh_shared_decode_workspace_size(B, c["Hs"], d, c["win"])), DEV)
        s["step_out"] = [{"topk_idx": torch.empty(B, K, dtype=torch.int32, device=DEV),
                          "gates": torch.empty(B, K, **f32),
                          "out": torch.empty(B, d, dtype=dt, device=DEV)}
                         for _ in range(c["steps"])]
    return s


# ---------------------------------------------------------------------------
# one pass

def _prefill(s, c):
    r = L.route(s["logits"], c["K"], out=s["r"], ws=s["rws"])
    fwd = L.attn_fwd_grouped if c["g"] > 1 else L.attn_fwd
    out = fwd(s["q"], s["k"], s["v"], r, c["K"], c["rope_base"], out=s["out"], ws=s["aws"])
    if c["Hs"]:
        L.shared_attn(s["qs"], s["ks"], s["vs"], c["win"], c["rope_base"], out=out,
                      accumulate=True, ws=s["sws"])
    return r, out


def _steps(s, c):
    """c["steps"] generated tokens of every sequence."""
    outs = []
    for i in range(c["steps"]):
        a = (s["step_logits"][i], s["step_q"][i], s["step_k"][i], s["step_v"][i], s["k_cache"],
             s["v_cache"], s["len"], c["K"], c["rope_base"])
        if c["g"] > 1:
            o = L.decode_step_grouped(*a, ws=s["dws"])
        else:
            o = L.decode_step(*a, out=s["step_out"][i], ws=s["dws"])
        if c["Hs"]:
            L.shared_decode_step(s["step_qs"][i], s["step_ks"][i], s["step_vs"][i], s["ks_cache"],
                                 s["vs_cache"], s["slen"], c["win"], c["rope_base"],
                                 out=o["out"], accumulate=True, ws=s["dsws"])
        outs.append(o)
    res = {"steps": outs, "k_cache": s["k_cache"], "v_cache": s["v_cache"], "len": s["len"]}
    if c["Hs"]:
        res.update(ks_cache=s["ks_cache"], vs_cache=s["vs_cache"], slen=s["slen"])
    return res


def run(state):
    s, c = state, state["c"]
    if c["kind"] == "prefill":
        r, out = _prefill(s, c)
        return {"out": out, "routing": r}
    if c["kind"] == "layer":
        r = L.route(s["logits"], c["K"], out=s["r"], ws=s["rws"])
        p = L.qkv_proj(s["x"], s["w_qkv"], r, c["H"], c["K"], out=s["qkv"])
        ho = L.attn_fwd(p["q"], p["k"], p["v"], r, c["K"], c["rope_base"], head_out=s["head_out"],
                        out=False, ws=s["aws"])
        out = L.out_proj(ho, s["w_o"], r, c["B"], c["T"], c["H"], c["K"], out=s["out"],
                         ws=s["ows"])
        return {"out": out, "head_out": ho, "gates": r["gates"], "topk_idx": r["topk_idx"]}
    if c["kind"] == "train":
        r = L.route(s["logits"], c["K"], out=s["r"], ws=s["rws"], bias=s.get("bias"))
        a = (s["q"], s["k"], s["v"], r, c["K"], c["rope_base"])
        if c["dtype"] == "bf16":
            out = L.attn_fwd_train(*a, s["bws"], out=s["out"])
        else:
            out = L.attn_fwd(*a, out=s["out"], ws=s["aws"])
        g = L.attn_bwd(*a, s["dout"], ws=s["bws"], out=s["grads"], packed=c["packed"],
                       saved=c["dtype"] == "bf16")
        mode = L.GATE_SOFTMAX_ALL if c["biased"] else L.GATE_SOFTMAX_SELECTED
        dl = L.route_bwd(s["logits"], r, g["dgates"], mode)
        return {"out": out, "grads": g, "dlogits": dl, "gates": r["gates"],
                "topk_idx": r["topk_idx"]}
    if c["kind"] == "decode":
        # the same tokens again from the same histories (a sampler that goes
        # back to a prefix sets the lengths back)
        s["len"].copy_(s["len0"])
        if c["Hs"]:
            s["slen"].copy_(s["slen0"])
        return _steps(s, c)
    r, out = _prefill(s, c)
    L.prefill_cache(s["k"], s["v"], r, c["K"], c["rope_base"], s["k_cache"], s["v_cache"],
                    s["len"])
    if c["Hs"]:
        L.shared_prefill_cache(s["ks"], s["vs"], s["ks_cache"], s["vs_cache"], s["slen"], c["win"],
                               c["rope_base"])
    return {"out": out, "gates": r["gates"], **_steps(s, c)}


# ---------------------------------------------------------------------------
# the same in 64 bits, in plain torch

def _rope64(x, pos, base):
    d = x.shape[-1]
    th = torch.pow(torch.tensor(float(base), dtype=torch.float64, device=x.device),
                   -2.0 * torch.arange(d // 2, dtype=torch.float64, device=x.device) / d)
    a = pos.to(torch.float64)[..., None] * th
    co, si = torch.cos(a), torch.sin(a)
    x1, x2 = x[..., :d // 2], x[..., d // 2:]
    return torch.cat([x1 * co - x2 * si, x2 * co + x1 * si], -1)


def _select64(c, logits, bias=None):
    """(topk [.., K], gates [.., K], gates over all heads [.., H])."""
    l64 = logits.double()
    aff = torch.softmax(l64, -1)
    score = logits if bias is None else (aff + bias.double()).float()
    top = torch.sort(score, dim=-1, descending=True, stable=True)[1][..., :c["K"]]
    if bias is None:
        return top, torch.softmax(l64.gather(-1, top), -1), aff
    return top, aff.gather(-1, top), aff


def _softmax_rows(q, k, lo, hi, scale, win=0):
    """P of the queries lo..hi of one head over its keys (causal)."""
    s = (q[lo:hi] @ k[:hi].T) * scale
    i = torch.arange(lo, hi, device=q.device)[:, None]
    j = torch.arange(hi, device=q.device)[None, :]
    s = s.masked_fill((j > i) | ((j <= i - win) if win else (j < 0)), float("-inf"))
    return torch.softmax(s, -1)


def _attend(q, k, v, scale, win=0):
    n, step = q.shape[0], 2048
    out = torch.empty_like(q)
    for lo in range(0, n, step):
        hi = min(n, lo + step)
        a = max(0, lo - win + 1) if win else 0
        p = _softmax_rows(q[a:], k[a:], lo - a, hi - a, scale, win)
        out[lo:hi] = p @ v[a:hi]
    return out


def _segments(c, top, gates):
    """(b, h, tokens, gates of those tokens, their k slots) of every head."""
    for b in range(c["B"]):
        for h in range(c["H"]):
            t, slot = torch.nonzero(top[b] == h, as_tuple=True)
            yield b, h, t, gates[b, t, slot], slot


def _prefill64(c, s, top, gates):
    out = torch.zeros(c["B"], c["T"], c["d"], dtype=torch.float64, device=DEV)
    scale, g, keys = c["d"] ** -0.5, c["g"], {}
    for b, h, t, gt, _ in _segments(c, top, gates):
        pos = torch.arange(len(t), device=DEV)
        k = _rope64(s["k"][b, h, t].double(), pos, c["rope_base"])
        v = s["v"][b, h, t].double()
        keys[b, h] = (k, v)
        for u in range(g):
            q = _rope64(s["q"][b, h * g + u, t].double(), pos, c["rope_base"])
            out[b, t] += gt[:, None] * _attend(q, k, v, scale)
    for i in range(c["Hs"]):
        pos = torch.arange(c["T"], device=DEV)
        for b in range(c["B"]):
            q, k = (_rope64(s[n][b, i].double(), pos, c["rope_base"]) for n in ("qs", "ks"))
            out[b] += _attend(q, k, s["vs"][b, i].double(), scale, c["win"])
    return out, keys


def _layer64(c, s):
    top, gates, _ = _select64(c, s["logits"])
    out = torch.zeros(c["B"], c["T"], c["dm"], dtype=torch.float64, device=DEV)
    heads = []
    for b, h, t, gt, _ in _segments(c, top, gates):
        x = s["x"][b, t].double()
        q, k, v = (x @ s["w_qkv"][h, i].double().T for i in range(3))
        pos = torch.arange(len(t), device=DEV)
        q, k = _rope64(q, pos, c["rope_base"]), _rope64(k, pos, c["rope_base"])
        o = _attend(q, k, v, c["d"] ** -0.5)
        heads.append(o)
        out[b, t] += (gt[:, None] * o) @ s["w_o"][h].double().T
    return {"out": out, "head_out": torch.cat(heads), "gates": gates, "topk_idx": None}


def _train64(c, s):
    B, T, H, K, d = (c[n] for n in ("B", "T", "H", "K", "d"))
    top, gates, aff = _select64(c, s["logits"], s.get("bias"))
    scale = d ** -0.5
    out = torch.zeros(B, T, d, dtype=torch.float64, device=DEV)
    dgates = torch.zeros(B, T, K, dtype=torch.float64, device=DEV)
    shape = (B * T * K, d) if c["packed"] else (B, H, T, d)
    dq, dk, dv = (torch.zeros(*shape, dtype=torch.float64, device=DEV) for _ in range(3))
    at = 0
    for b, h, t, gt, slot in _segments(c, top, gates):
        n = len(t)
        pos = torch.arange(n, device=DEV)
        q, k = (_rope64(s[m][b, h, t].double(), pos, c["rope_base"]) for m in ("q", "k"))
        v, do = s["v"][b, h, t].double(), s["dout"][b, t].double()
        go = gt[:, None] * do
        gq, gk, gv = torch.zeros_like(q), torch.zeros_like(q), torch.zeros_like(q)
        for lo in range(0, n, 2048):
            hi = min(n, lo + 2048)
            p = _softmax_rows(q, k, lo, hi, scale)
            o = p @ v[:hi]
            out[b, t[lo:hi]] += gt[lo:hi, None] * o
            dgates[b, t[lo:hi], slot[lo:hi]] = (o * do[lo:hi]).sum(-1)
            gv[:hi] += p.T @ go[lo:hi]
            ds = p * (go[lo:hi] @ v[:hi].T - (go[lo:hi] * o).sum(-1, keepdim=True)) * scale
            gq[lo:hi] = ds @ k[:hi]
            gk[:hi] += ds.T @ q[lo:hi]
        gq, gk = (_rope64(x, -pos, c["rope_base"]) for x in (gq, gk))
        for dst, x in ((dq, gq), (dk, gk), (dv, gv)):
            if c["packed"]:
                dst[at:at + n] = x
            else:
                dst[b, h, t] = x
        at += n
    if c["biased"]:
        da = torch.zeros(B, T, H, dtype=torch.float64, device=DEV).scatter_(-1, top, dgates)
        dl = aff * (da - (aff * da).sum(-1, keepdim=True))
    else:
        part = gates * (dgates - (gates * dgates).sum(-1, keepdim=True))
        dl = torch.zeros(B, T, H, dtype=torch.float64, device=DEV).scatter_(-1, top, part)
    return {"out": out, "grads": {"dq": dq, "dk": dk, "dv": dv, "dgates": dgates}, "dlogits": dl,
            "gates": gates, "topk_idx": None}


def _steps64(c, s, rows, srows):
    """rows(b, h): the head's cached (keys, values) in float64, rotated;
    srows(b, i): the shared head's history likewise, with its next position."""
    d, scale, g = c["d"], c["d"] ** -0.5, c["g"]
    new, snew, res = {}, {}, []

    def attend(q, k, v):
        return torch.softmax((k @ q) * scale, 0) @ v

    for i in range(c["steps"]):
        top, gates, _ = _select64(c, s["step_logits"][i])
        picks = top.cpu().tolist()
        out = torch.zeros(c["B"], d, dtype=torch.float64, device=DEV)
        for b in range(c["B"]):
            for j, h in enumerate(picks[b]):
                if (b, h) not in new:
                    new[b, h] = rows(b, h)
                k, v = new[b, h]
                pos = torch.tensor(k.shape[0], device=DEV)
                kn = _rope64(s["step_k"][i, b, h].double(), pos, c["rope_base"])
                k, v = torch.cat([k, kn[None]]), torch.cat([v, s["step_v"][i, b, h].double()[None]])
                new[b, h] = (k, v)
                for u in range(g):
                    q = _rope64(s["step_q"][i, b, h * g + u].double(), pos, c["rope_base"])
                    out[b] += gates[b, j] * attend(q, k, v)
            for m in range(c["Hs"]):
                if (b, m) not in snew:
                    snew[b, m] = srows(b, m)
                k, v, p = snew[b, m]
                pos = torch.tensor(p, device=DEV)
                kn = _rope64(s["step_ks"][i, b, m].double(), pos, c["rope_base"])
                k = torch.cat([k, kn[None]])[-c["win"]:]
                v = torch.cat([v, s["step_vs"][i, b, m].double()[None]])[-c["win"]:]
                snew[b, m] = (k, v, p + 1)
                q = _rope64(s["step_qs"][i, b, m].double(), pos, c["rope_base"])
                out[b] += attend(q, k, v)
        res.append({"topk_idx": None, "gates": gates, "out": out})
    return res, new


def _caches64(c, base, lens, new):
    """The caches after the steps, float64."""
    k, v = (x.double() for x in base)
    for (b, h), (kr, vr) in new.items():
        n = kr.shape[0]
        lo = int(lens[b][h])
        k[b, h, lo:n], v[b, h, lo:n] = kr[lo:], vr[lo:]
    return k, v


def exact(case, seed):
    c = case
    s = _inputs(c, _gen(seed))
    with torch.no_grad():
        if c["kind"] == "prefill":
            top, gates, _ = _select64(c, s["logits"])
            ints = ("topk_idx", "head_len", "seg_offsets", "perm_token", "slot_pos")
            return {"out": _prefill64(c, s, top, gates)[0],
                    "routing": dict({n: None for n in ints}, gates=gates)}
        if c["kind"] == "layer":
            return _layer64(c, s)
        if c["kind"] == "train":
            return _train64(c, s)
        shared = {"ks_cache": None, "vs_cache": None, "slen": None} if c["Hs"] else {}
        if c["kind"] == "decode":
            lens = s["len0"].cpu().tolist()

            def rows(b, h):
                return tuple(s[n][b, h, :lens[b][h]].double() for n in ("k_cache", "v_cache"))

            def srows(b, i):
                w, p = c["win"], c["prior"]
                m = min(p, w)
                idx = torch.arange(p - m, p, device=DEV) % w
                return (*(s[n][b, i, idx].double() for n in ("ks_cache", "vs_cache")), p)

            steps, new = _steps64(c, s, rows, srows)
            res = {"steps": steps, "k_cache": None, "v_cache": None, "len": None, **shared}
            if s["k_cache"].numel() <= 1 << 28:
                res["k_cache"], res["v_cache"] = _caches64(c, (s["k_cache"], s["v_cache"]), lens,
                                                           new)
            return res
        top, gates, _ = _select64(c, s["logits"])
        out, keys = _prefill64(c, s, top, gates)
        lens = [[0] * c["H"] for _ in range(c["B"])]

        def srows(b, i):
            pos = torch.arange(c["T"], device=DEV)
            k = _rope64(s["ks"][b, i].double(), pos, c["rope_base"])
            return k[-c["win"]:], s["vs"][b, i, -c["win"]:].double(), c["T"]

        steps, new = _steps64(c, s, lambda b, h: keys[b, h], srows)
        k, v = _caches64(c, (s["k_cache"], s["v_cache"]), lens, {**keys, **new})
        return {"out": out, "gates": gates, "steps": steps, "k_cache": k, "v_cache": v,
                "len": None, **shared}
