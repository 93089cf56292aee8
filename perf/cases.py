"""Performance cases: the calls a serving engine or a trainer makes through ``paper_2605_06676_amd.lkv``.

Each case is one pass through public entry points on inputs drawn from a seed.  The listed cases cover

* scoring of a prefilled cache (linear scorer over ragged prompts; the 256-128-1 SiLU scorer, one per head),
* top-k + compaction of a whole cache with planned offsets,
* eviction of one layer during prefill (short heads; long heads with counted scores and a split top-k),
* the observation-window scorer,
* decode attention over the packed cache (all layers at once; one small layer),
* training-time attention with the multiplicative mask (forward, backward, and both for a short odd length),
* the batched Soft-TopK of a training sample, forward and backward.

Shapes are those of ``workloads.CONFIGS``, of the tests and of ``bench.py``; ``draw`` spreads them.
"""
import math

import numpy as np
import torch

from paper_2605_06676_amd import lkv
from paper_2605_06676_amd import workloads as W

D = 128
_DEVICE = "cuda:0"
_ctx = None


def _context():
    """The process's library context (a program makes one and keeps it)."""
    global _ctx
    if _ctx is None:
        _ctx = lkv.Context(0)
    return _ctx


def listed():
    return [
        # one layer of one decode step on a short prompt: launches and their latency are all there is
        {"name": "decode-layer-4k", "op": "decode", "n_seq": 1, "L": 1, "H": 8, "G": 4, "T": 4096, "R": 0.15},
        # one decode step over the packed caches of all layers of a 32k prompt (8B-class model shape)
        {"name": "decode-32k", "op": "decode", "n_seq": 1, "L": 32, "H": 8, "G": 4, "T": 32768, "R": 0.15},
        # linear scorer over a batch of prompts of different, odd lengths
        {"name": "score-linear-ragged", "op": "score", "n_seq": 4, "ragged": True, "L": 32, "H": 8, "T": 16384,
         "hidden": 0, "act": "silu", "per_head": False},
        # the paper's scorer (256-128-1 SiLU, one per head) over a 32k prompt
        {"name": "score-mlp128-32k", "op": "score", "n_seq": 1, "ragged": False, "L": 32, "H": 8, "T": 32768,
         "hidden": 128, "act": "silu", "per_head": True},
        # top-k and compaction of a whole 32k cache, offsets planned beforehand
        {"name": "select-compact-32k", "op": "select", "n_seq": 1, "L": 32, "H": 8, "T": 32768, "R": 0.15},
        # a layer evicted as soon as the prefill has produced it: linear scorer, 32k prompt
        {"name": "evict-layer-32k", "op": "evict_layer", "n_seq": 1, "m": 1, "H": 8, "T": 32768, "R": 0.15,
         "hidden": 0, "act": "silu", "counted": False},
        # the same at 128k with the 256-64-1 GELU scorer, counted scores and room for the split top-k
        {"name": "evict-layer-128k", "op": "evict_layer", "n_seq": 1, "m": 1, "H": 8, "T": 131072, "R": 0.10,
         "hidden": 64, "act": "gelu", "counted": True},
        # observation-window scorer over a whole 32k cache, normalisers not supplied
        {"name": "window-32k", "op": "window", "n_seq": 1, "L": 32, "H": 8, "G": 4, "T": 32768, "window": 32,
         "pool_width": 7, "pool_max": True, "given_lse": False},
        # training-time attention of one layer at the longest sample length, each direction
        {"name": "attn-fwd-16k", "op": "attn_fwd", "H": 8, "G": 4, "T": 16384},
        {"name": "attn-bwd-16k", "op": "attn_bwd", "H": 8, "G": 4, "T": 16384},
        # both directions of a short sample of odd length
        {"name": "attn-train-2k", "op": "attn_train", "H": 8, "G": 4, "T": 2345},
        # the soft masks of all heads of a training sample and their gradients
        {"name": "soft-topk-16k", "op": "soft_topk", "n_vec": 256, "n": 16384, "tau": 0.1, "f64": False},
    ]


def _log_int(rng, lo, hi):
    """A whole number in [lo, hi], spread over its logarithm; odd in half of the draws."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        v |= 1
    return max(lo, min(hi, v))


def draw(rng):
    op = rng.choice(["decode", "decode", "score", "select", "evict_layer", "window", "attn_fwd", "attn_bwd", "attn_train",
                     "soft_topk"])
    H, G = rng.choice([(8, 4), (8, 4), (4, 7), (2, 8), (8, 1)])
    if op == "decode":
        L = rng.choice([1, 1, 8, 32])
        n_seq = rng.choice([1, 1, 2, 8])
        return {"op": op, "n_seq": n_seq, "L": L, "H": H, "G": G, "T": _log_int(rng, 2048, 131072 // (L * n_seq) + 4096),
                "R": rng.choice([0.05, 0.1, 0.15])}
    if op == "score":
        kind = rng.choice([(0, "silu", False), (64, "gelu", False), (128, "silu", True), (64, "silu", True)])
        n_seq = rng.choice([1, 1, 3])
        L = rng.choice([1, 8, 32])
        return {"op": op, "n_seq": n_seq, "ragged": n_seq > 1, "L": L, "H": H,
                "T": _log_int(rng, 4096, min(131072, 32 * 32768 // (L * n_seq))),
                "hidden": kind[0], "act": kind[1], "per_head": kind[2]}
    if op == "select":
        L = rng.choice([1, 8, 32])
        return {"op": op, "n_seq": 1, "L": L, "H": H, "T": _log_int(rng, 4096, min(131072, 32 * 32768 // L)),
                "R": rng.choice([0.05, 0.1, 0.15])}
    if op == "evict_layer":
        T = _log_int(rng, 4096, 131072)
        hidden, act = rng.choice([(0, "silu"), (64, "gelu"), (128, "silu")])
        return {"op": op, "n_seq": rng.choice([1, 1, 2]), "m": rng.choice([1, 1, 2, 4]), "H": H, "T": T,
                "R": rng.choice([0.05, 0.1, 0.15]), "hidden": hidden, "act": act, "counted": rng.random() < 0.5}
    if op == "window":
        L = rng.choice([1, 8, 32])
        return {"op": op, "n_seq": 1, "L": L, "H": H, "G": G, "T": _log_int(rng, 4096, min(131072, 32 * 32768 // L)),
                "window": rng.choice([8, 16]) if G > 4 else rng.choice([8, 16, 32]), "pool_width": rng.choice([1, 5, 7, 13]),
                "pool_max": rng.random() < 0.7, "given_lse": rng.random() < 0.4}
    if op == "soft_topk":
        n = _log_int(rng, 512, 32768)
        return {"op": op, "n_vec": rng.choice([1, 8, 32, 256]), "n": n, "tau": rng.choice([0.02, 0.1, 0.5, 1.0]),
                "f64": rng.random() < 0.3 and n <= 16384}
    if op == "attn_train":
        return {"op": op, "H": H, "G": G, "T": _log_int(rng, 1024, 8192)}
    return {"op": op, "H": H, "G": G, "T": _log_int(rng, 2048, 16384)}


# ---- inputs -------------------------------------------------------------------------------------


def _gen(seed, tag):
    g = torch.Generator(device=_DEVICE)
    g.manual_seed(int(seed) * 64 + tag)
    return g


def _normal(shape, seed, tag, dtype=torch.bfloat16):
    return torch.empty(shape, dtype=dtype, device=_DEVICE).normal_(generator=_gen(seed, tag))


def _uniform(shape, seed, tag):
    return torch.rand(shape, dtype=torch.float32, device=_DEVICE, generator=_gen(seed, tag))


def _lengths(case):
    """Sequence lengths: fixed by the case, not by the seed, so that every seed is the same amount of work."""
    n, T = case["n_seq"], case["T"]
    if not case.get("ragged"):
        return [T] * n
    return [T - ((T * 3 // 4) * i // max(1, n - 1)) - (37 * i) % 64 for i in range(n)]


def _kv(case, L, seed):
    """Per-sequence K and V, bf16 [L, H, T_s, 128], i.i.d. normal with a few x10 outlier channels."""
    k, v = [], []
    for s, T in enumerate(_lengths(case)):
        for i, dst in enumerate((k, v)):
            x = _normal((L, case["H"], T, D), seed, 2 * s + i)
            ch = torch.randint(0, D, (2,), generator=_gen(seed, 40 + i), device=_DEVICE)
            x[..., ch] *= 10.0
            dst.append(x)
    return k, v


def _scorer(case, L, seed):
    hidden = case["hidden"]
    w = W.scaled(W.CONFIGS[0], L=L, H=case["H"], scorer="mlp" if hidden else "linear", hidden=hidden, act=case["act"],
                 per_head=bool(case.get("per_head", False)), out_bias=not case.get("per_head", False))
    s = W.draw_scorer(w, seed)
    s["w1"] = torch.from_numpy(s["w1"].view(np.int16)).to(_DEVICE).view(torch.bfloat16)
    for name in ("b1", "w2", "b2"):
        if s[name] is not None:
            s[name] = torch.from_numpy(s[name]).to(_DEVICE)
    return s


def _budgets(case, L, seed):
    """Skewed budgets of every head (Dirichlet shares over the flattened heads), host int32 [n_seq * L * H].  The shares
    are one fixed table, dealt to the heads in an order that the seed turns, so that every seed keeps as many rows."""
    w = W.scaled(W.CONFIGS[1], L=L, H=case["H"], Hq=case["H"], T=case["T"], R=case["R"], n_seq=case["n_seq"], b_min=32)
    return np.concatenate([np.roll(W.draw_budgets(w, T, i).reshape(-1), seed) for i, T in enumerate(_lengths(case))])


def _plan(ctx, budgets):
    offsets = torch.empty(budgets.size + 1, dtype=torch.int32, device=_DEVICE)
    return offsets, lkv.lkv_plan_offsets(ctx, budgets, offsets)


def _attn_inputs(case, seed):
    H, Hq, T = case["H"], case["H"] * case["G"], case["T"]
    x = _uniform((H, T), seed, 4)
    m = x ** 4                                        # most weights small, some exactly 0 and 1
    pick = _uniform((H, T), seed, 5)
    m[pick < 0.10] = 0.0
    m[pick > 0.95] = 1.0
    m[:, 0] = m[:, 0].clamp(min=0.25)                 # every causal prefix carries weight
    return {"q": _normal((Hq, T, D), seed, 0), "k": _normal((H, T, D), seed, 1), "v": _normal((H, T, D), seed, 2), "m": m,
            "d_o": _normal((Hq, T, D), seed, 3)}


def _attn_buffers(case):
    H, Hq, T = case["H"], case["H"] * case["G"], case["T"]
    f = dict(dtype=torch.float32, device=_DEVICE)
    ws = lkv.lkv_masked_attn_backward_workspace_bytes(Hq, H, T)
    return {"o": torch.empty((Hq, T, D), **f), "lse": torch.empty((Hq, T), **f), "dq": torch.empty((Hq, T, D), **f),
            "dk": torch.empty((H, T, D), **f), "dv": torch.empty((H, T, D), **f), "dm": torch.empty((H, T), **f),
            "ws": torch.empty(ws, dtype=torch.uint8, device=_DEVICE)}


def _window_inputs(case, seed):
    """Keys and window queries; half of the query rows lean towards one of a few planted keys of the prefix."""
    L, H, G, T, Wn = case["L"], case["H"], case["G"], case["T"], case["window"]
    k = _normal((L, H, T, D), seed, 0)
    q = _normal((L, H, G, Wn, D), seed, 1, torch.float32)
    needles = torch.randint(0, T - Wn, (L, H, G, 4), generator=_gen(seed, 2), device=_DEVICE)
    which = torch.randint(0, 4, (L, H, G, Wn), generator=_gen(seed, 3), device=_DEVICE)
    pos = torch.gather(needles, 3, which).reshape(L, H, G * Wn, 1).expand(-1, -1, -1, D)
    rows = torch.gather(k, 2, pos).reshape(L, H, G, Wn, D).float()
    planted = (_uniform((L, H, G, Wn, 1), seed, 4) < 0.5).float()
    q = (q + 0.5 * rows * planted).to(torch.bfloat16).reshape(L, H * G, Wn, D).contiguous()
    return k, q


def _window_logits(case, k, q, l, h):
    """fp64 logits [G * W, T] of one head, -inf on the keys a window row does not see."""
    G, T, Wn = case["G"], case["T"], case["window"]
    s = q[l, h * G:(h + 1) * G].reshape(G * Wn, D).double() @ k[l, h].double().T / math.sqrt(D)
    i = torch.arange(Wn, device=_DEVICE).repeat(G)
    return s.masked_fill(torch.arange(T, device=_DEVICE)[None, :] > (T - Wn + i)[:, None], -math.inf)


def _topk_inputs(case, seed):
    """Noisy scores of a sample's heads, their target sums (a wide spread of ratios) and an upstream gradient."""
    n_vec, n = case["n_vec"], case["n"]
    dtype = torch.float64 if case["f64"] else torch.float32
    u = _normal((n_vec, n), seed, 0, torch.float32) * 0.5
    e = _uniform((n_vec, n), seed, 1).clamp(1e-6, 1.0 - 1e-6)
    x = (u - torch.log(-torch.log(e))).to(dtype)
    k = (0.02 + 0.5 * _uniform((n_vec,), seed, 2).double() ** 2) * n
    return x, k, _normal((n_vec, n), seed, 3, torch.float32).double()


def prepare(case, seed):
    ctx, op = _context(), case["op"]
    s = {"op": op, "case": case, "ctx": ctx}
    f32 = dict(dtype=torch.float32, device=_DEVICE)
    if op == "decode":
        n_seg, Hq = case["n_seq"] * case["L"] * case["H"], case["H"] * case["G"]
        s["offsets"], total = _plan(ctx, _budgets(case, case["L"], seed))
        s["total"] = total
        s["kp"], s["vp"] = _normal((total, D), seed, 0), _normal((total, D), seed, 1)
        s["q"] = _normal((case["n_seq"], case["L"], Hq, D), seed, 2)
        s["out"] = torch.empty((case["n_seq"], case["L"], Hq, D), **f32)
        s["lse"] = torch.empty((case["n_seq"], case["L"], Hq), **f32)
        ws = lkv.lkv_decode_workspace_bytes(n_seg, total, Hq, case["H"])
        s["ws"] = torch.empty(ws, dtype=torch.uint8, device=_DEVICE)
    elif op in ("score", "select", "evict_layer"):
        L = case["m"] if op == "evict_layer" else case["L"]
        k, v = _kv(case, L, seed)
        s["cache"] = lkv.Cache(k, v, case["H"] * 4)
        lens = _lengths(case)
        if op == "select":   # scores shaped like a trained scorer's: a heavy-tailed mixture with ties
            s["scores"] = [_normal((L, case["H"], T), seed, 20 + i, torch.float32) * 0.3 for i, T in enumerate(lens)]
            for x in s["scores"]:
                x[..., ::61] = x[..., ::61].to(torch.bfloat16).float()
        else:
            s["scores"] = [torch.empty((L, case["H"], T), **f32) for T in lens]
            s["scorer"] = _scorer(case, L, seed)
        if op != "score":
            s["budgets"] = _budgets(case, L, seed)
            s["offsets"], total = _plan(ctx, s["budgets"])
            s["total"] = total
            s["idx"] = torch.empty(total, dtype=torch.int32, device=_DEVICE)
            s["kp"] = torch.empty((total, D), dtype=torch.bfloat16, device=_DEVICE)
            s["vp"] = torch.empty((total, D), dtype=torch.bfloat16, device=_DEVICE)
        s["counts"] = None
        if case.get("counted"):
            n_seg = case["n_seq"] * L * case["H"]
            s["counts"] = torch.empty(lkv.lkv_counts_bytes_split(n_seg, max(lens)), dtype=torch.uint8, device=_DEVICE)
            lkv.lkv_clear_counts(ctx, s["counts"], n_seg)
    elif op == "window":
        k, q = _window_inputs(case, seed)
        s["cache"] = lkv.Cache([k], [k], case["H"] * case["G"])   # the value cache is not read
        s["q"] = [q]
        s["scores"] = [torch.empty((case["L"], case["H"], case["T"]), **f32)]
        s["ws"] = torch.empty(lkv.lkv_score_window_workspace_bytes(s["cache"]), dtype=torch.uint8, device=_DEVICE)
        s["lse"] = None
        if case["given_lse"]:   # what the prefill's attention kernel left for these queries
            lse = torch.empty((case["L"], case["H"], case["G"] * case["window"]), **f32)
            for l in range(case["L"]):
                for h in range(case["H"]):
                    lse[l, h] = torch.logsumexp(_window_logits(case, k, q, l, h).float(), dim=1)
            s["lse"] = [lse.reshape(case["L"], case["H"] * case["G"], case["window"])]
    elif op in ("attn_fwd", "attn_bwd", "attn_train"):
        s.update(_attn_inputs(case, seed))
        s.update(_attn_buffers(case))
        if op == "attn_bwd":   # the backward pass starts from what the forward pass returned
            _attn_forward(s)
    else:
        s["x"], s["k"], s["g"] = _topk_inputs(case, seed)
        f64 = dict(dtype=torch.float64, device=_DEVICE)
        s["y"], s["dx"] = torch.empty(s["x"].shape, **f64), torch.empty(s["x"].shape, **f64)
        s["info"], s["dk"] = torch.empty((case["n_vec"], 2), **f64), torch.empty(case["n_vec"], **f64)
    return s


# ---- one pass -----------------------------------------------------------------------------------


def _attn_forward(s):
    lkv.lkv_masked_attn_forward(s["ctx"], s["q"], s["k"], s["v"], s["m"], 1.0 / math.sqrt(D), s["o"], s["lse"])


def _attn_backward(s):
    lkv.lkv_masked_attn_backward(s["ctx"], s["q"], s["k"], s["v"], s["m"], s["o"], s["lse"], s["d_o"], 1.0 / math.sqrt(D),
                                 s["dq"], s["dk"], s["dv"], s["dm"], s["ws"])


def run(s):
    ctx, op, case = s["ctx"], s["op"], s["case"]
    if op == "decode":
        lkv.lkv_decode_attn(ctx, case["n_seq"], case["L"], case["H"], case["H"] * case["G"], D, s["q"], s["kp"], s["vp"],
                            s["offsets"], s["total"], 1.0 / math.sqrt(D), s["out"], s["lse"], s["ws"])
        return {"out": s["out"], "lse": s["lse"]}
    if op == "score":
        lkv.lkv_score(ctx, s["cache"], s["scorer"], s["scores"])
        return {"scores": s["scores"]}
    if op == "select":
        lkv.lkv_select(ctx, s["cache"], s["scores"], None, s["idx"], s["offsets"])
        lkv.lkv_compact(ctx, s["cache"], s["idx"], s["offsets"], s["total"], s["kp"], s["vp"])
        return {"idx": s["idx"], "kp": s["kp"], "vp": s["vp"]}
    if op == "evict_layer":
        lkv.lkv_evict_layer(ctx, s["cache"], 0, case["m"], s["scorer"], s["budgets"], s["offsets"], s["scores"], s["idx"],
                            s["kp"], s["vp"], counts=s["counts"])
        return {"scores": s["scores"], "idx": s["idx"], "kp": s["kp"], "vp": s["vp"]}
    if op == "window":
        lkv.lkv_score_window(ctx, s["cache"], s["q"], case["window"], case["pool_width"],
                             lkv.POOL_MAX if case["pool_max"] else lkv.POOL_AVG, 1.0 / math.sqrt(D), s["scores"], s["ws"],
                             lse_win=s["lse"])
        return {"scores": s["scores"]}
    if op == "soft_topk":
        lkv.lkv_soft_topk_batched(ctx, s["x"], s["k"], case["tau"], s["y"], s["info"])
        lkv.lkv_soft_topk_backward_batched(ctx, s["x"], case["tau"], s["info"], s["g"], s["dx"], s["dk"])
        return {"y": s["y"], "info": s["info"], "dx": s["dx"], "dk": s["dk"]}
    out = {}
    if op != "attn_bwd":
        _attn_forward(s)
        out.update(o=s["o"], lse=s["lse"])
    if op != "attn_fwd":
        _attn_backward(s)
        out.update(dq=s["dq"], dk=s["dk"], dv=s["dv"], dm=s["dm"])
    return out


# ---- what a pass cannot do without --------------------------------------------------------------


def _kept(case, L):
    return case["R"] * case["H"] * L * sum(_lengths(case))


def work(case):
    op = case["op"]
    if op == "decode":
        rows, heads = _kept(case, case["L"]), case["n_seq"] * case["L"] * case["H"] * case["G"]
        return {"bytes": rows * 512 + heads * (256 + 512 + 4), "flops": 4.0 * D * rows * case["G"]}
    if op in ("score", "select", "evict_layer"):
        L = case["m"] if op == "evict_layer" else case["L"]
        tokens = case["H"] * L * sum(_lengths(case))
        if op == "select":
            return {"bytes": tokens * 4 + _kept(case, L) * (4 + 1024), "flops": 0}
        hidden = case["hidden"]
        flops = tokens * (2.0 * 256 * max(1, hidden) + 2 * hidden)
        if op == "score":
            return {"bytes": tokens * (512 + 4), "flops": flops}
        return {"bytes": tokens * (512 + 4) + _kept(case, L) * (4 + 512), "flops": flops}
    if op == "window":
        keys, rows = case["L"] * case["H"] * case["T"], case["G"] * case["window"]
        return {"bytes": keys * (256 + 4) + case["L"] * case["H"] * rows * 256, "flops": 2.0 * D * rows * keys}
    if op == "soft_topk":
        n = case["n_vec"] * case["n"]
        size = 8 if case["f64"] else 4
        # forward: x in, y out; backward: x and g in, dx out
        return {"bytes": n * (size + 8) + n * (size + 16), "flops": 0}
    H, Hq, T = case["H"], case["H"] * case["G"], case["T"]
    product = D * float(T) * (T + 1) * Hq               # one product over the causal triangle
    read = (Hq + 2 * H) * T * D * 2 + H * T * 4         # q, k, v, m
    fwd = {"bytes": read + Hq * T * (D * 4 + 4), "flops": 2 * product}
    bwd = {"bytes": read + Hq * T * (D * 4 + 4 + D * 2) + (Hq + 2 * H) * T * D * 4 + H * T * 4, "flops": 5 * product}
    if op == "attn_fwd":
        return fwd
    if op == "attn_bwd":
        return bwd
    return {x: fwd[x] + bwd[x] for x in fwd}


def tolerance(case):
    """About four times what two correct implementations were seen to differ by (each against ``exact``)."""
    op = case["op"]
    if op == "select":
        return "exact"                                       # whole numbers and copied rows
    if op in ("score", "evict_layer"):
        # fp32 sums of exact products, seen at 6e-8 to 6e-7; kept tokens change only where two scores next to the
        # threshold agree to the last bits
        return {"rel": 3e-6, "max": 2e-4, "differ": 0.01}
    if op == "window":
        return {"rel": 3e-6, "max": 2e-4}                    # fp32 softmax, seen at 5e-7
    if op == "soft_topk":
        return {"rel": 1e-11, "max": 1e-9}                   # fp64 throughout, seen at 1e-15 to 1e-13
    if op == "decode":
        return {"rel": 5e-3, "max": 0.2}                     # probabilities rounded to bf16, seen at 1.2e-3
    # bf16 probabilities and gradient factors, seen at 1.7e-3; single early rows are differences of nearly equal numbers
    return {"rel": 7e-3, "max": 0.5}


# ---- the same numbers in 64 bits ----------------------------------------------------------------


def _exact_scores(case, seed):
    L = case["m"] if case["op"] == "evict_layer" else case["L"]
    k, v = _kv(case, L, seed)
    p = _scorer(case, L, seed)
    act = torch.nn.functional.silu if case["act"] == "silu" else torch.nn.functional.gelu
    out = []
    for K, V in zip(k, v):
        u = torch.empty(K.shape[:3], dtype=torch.float64, device=_DEVICE)
        for l in range(L):
            for h in range(case["H"]):
                hs = h if p["per_head"] else 0
                x = torch.cat([K[l, h], V[l, h]], dim=1).double()
                z = x @ p["w1"][l, hs].double().T + p["b1"][l, hs].double()
                if case["hidden"]:
                    z = act(z) @ p["w2"][l, hs].double()
                    if p["b2"] is not None:
                        z = z + p["b2"][l, hs].double()
                u[l, h] = z
        out.append(u)
    return out


def _exact_decode(case, seed):
    b = _budgets(case, case["L"], seed)
    off = np.concatenate([[0], np.cumsum(b)])
    total, G = int(off[-1]), case["G"]
    Hq = case["H"] * G
    kp, vp = _normal((total, D), seed, 0), _normal((total, D), seed, 1)
    q = _normal((case["n_seq"], case["L"], Hq, D), seed, 2).double().reshape(b.size, G, D)
    out = torch.zeros((b.size, G, D), dtype=torch.float64, device=_DEVICE)
    lse = torch.full((b.size, G), -math.inf, dtype=torch.float64, device=_DEVICE)
    for i in range(b.size):
        if b[i] > 0:
            sc = q[i] @ kp[off[i]:off[i + 1]].double().T / math.sqrt(D)
            lse[i] = torch.logsumexp(sc, dim=1)
            out[i] = torch.softmax(sc, dim=1) @ vp[off[i]:off[i + 1]].double()
    shape = (case["n_seq"], case["L"], Hq)
    return {"out": out.reshape(shape + (D,)), "lse": lse.reshape(shape)}


def _exact_window(case, seed):
    k, q = _window_inputs(case, seed)
    L, H, G, T, Wn = case["L"], case["H"], case["G"], case["T"], case["window"]
    c = (case["pool_width"] - 1) // 2
    out = torch.full((L, H, T), math.inf, dtype=torch.float64, device=_DEVICE)
    for l in range(L):
        for h in range(H):
            vote = torch.softmax(_window_logits(case, k, q, l, h), dim=1).sum(dim=0)[:T - Wn] / G
            if case["pool_max"]:
                pooled = torch.nn.functional.max_pool1d(vote[None, None], 2 * c + 1, stride=1, padding=c)
            else:
                pooled = torch.nn.functional.avg_pool1d(vote[None, None], 2 * c + 1, stride=1, padding=c)
            out[l, h, :T - Wn] = pooled[0, 0]
    return {"scores": [out]}


def _exact_attn(case, seed):
    x = _attn_inputs(case, seed)
    H, G, T, op = case["H"], case["G"], case["T"], case["op"]
    f64 = dict(dtype=torch.float64, device=_DEVICE)
    out = {}
    if op != "attn_bwd":
        out.update(o=torch.empty((H * G, T, D), **f64), lse=torch.empty((H * G, T), **f64))
    if op != "attn_fwd":
        out.update(dq=torch.empty((H * G, T, D), **f64), dk=torch.zeros((H, T, D), **f64), dv=torch.zeros((H, T, D), **f64),
                   dm=torch.zeros((H, T), **f64))
    scale = 1.0 / math.sqrt(D)
    step = 4096                                              # query rows at a time
    for hq in range(H * G):
        h = hq // G
        k, v, m = x["k"][h].double(), x["v"][h].double(), x["m"][h].double()
        for i0 in range(0, T, step):
            i1 = min(T, i0 + step)
            q = x["q"][hq, i0:i1].double()
            s = q @ k[:i1].T * scale
            s = s.masked_fill_(torch.arange(i1, device=_DEVICE)[None, :] > torch.arange(i0, i1, device=_DEVICE)[:, None], -math.inf)
            top = s.amax(dim=1, keepdim=True)
            e = torch.exp(s - top)
            z = e @ m[:i1, None]
            e /= z
            p = e * m[None, :i1]
            o = p @ v[:i1]
            if op != "attn_bwd":
                out["o"][hq, i0:i1], out["lse"][hq, i0:i1] = o, (top + torch.log(z))[:, 0]
            if op != "attn_fwd":
                g = x["d_o"][hq, i0:i1].double()
                out["dv"][h, :i1] += p.T @ g
                diff = g @ v[:i1].T - (g * o).sum(dim=1, keepdim=True)
                out["dm"][h, :i1] += (e * diff).sum(dim=0)
                ds = p * diff * scale
                out["dq"][hq, i0:i1] = ds @ k[:i1]
                out["dk"][h, :i1] += ds.T @ q
    return out


def _exact_soft_topk(case, seed):
    x, k, g = _topk_inputs(case, seed)
    n, tau = case["n"], case["tau"]
    z = x.double() / tau
    k = k.clamp(1e-6, n - 1e-6)
    v = torch.sort(z, dim=1, descending=True).values
    top, low = v[:, :1], v[:, -1:]
    # sums over the head and the tail at every split, each relative to its own largest exponent
    s1 = torch.logcumsumexp(-v, dim=1)
    s2 = torch.flip(torch.logcumsumexp(torch.flip(v, (1,)), dim=1), (1,))
    none = torch.full_like(top, -math.inf)
    s1, s2 = torch.cat([none, s1], 1), torch.cat([s2, none], 1)     # index m = values in the head
    rank = torch.arange(1, n + 1, device=_DEVICE, dtype=torch.float64)[None, :]
    at = rank - k[:, None] - 0.5 * torch.exp(v + s1[:, 1:]) + 0.5 * torch.exp(s2[:, 1:] - v)
    m = (at <= 0).sum(dim=1)
    a, b = s1.gather(1, m[:, None])[:, 0], s2.gather(1, m[:, None])[:, 0]
    d = k - m
    h = 0.5 * (a + b)
    root = torch.where(torch.isfinite(h), h + torch.asinh(d.abs() * torch.exp(-h)), torch.log(2.0 * d.abs()))
    lam = torch.where(d >= 0, b - root, root - a)
    t = z - lam[:, None]
    y = torch.where(t >= 0, 1.0 - 0.5 * torch.exp(-t.abs()), 0.5 * torch.exp(-t.abs()))
    slope = 0.5 * torch.exp(-t.abs())
    rel = torch.exp(t.abs().amin(dim=1, keepdim=True) - t.abs())
    dk = (g * rel).sum(dim=1) / rel.sum(dim=1)
    return {"y": y, "info": torch.stack([lam, m.double()], 1), "dx": slope / tau * (g - dk[:, None]), "dk": dk}


def exact(case, seed):
    op = case["op"]
    if op == "select":
        return None                                          # positions and copies, compared as they are
    if op == "score":
        return {"scores": _exact_scores(case, seed)}
    if op == "evict_layer":
        return {"scores": _exact_scores(case, seed), "idx": None, "kp": None, "vp": None}
    if op == "decode":
        return _exact_decode(case, seed)
    if op == "window":
        return _exact_window(case, seed)
    if op == "soft_topk":
        return _exact_soft_topk(case, seed)
    return _exact_attn(case, seed)
