"""The calls whose speed matters to a user of this library, over the sizes they are made at.

Six kinds, each through the binding as a decoding loop uses it:
  attention   one layer's tree attention: bf16, fp32 or an fp8 prefix cache; all tree rows or the newest level only;
              one key/value head per query head or several query heads sharing one
  step        one verification step of a whole model: mask slice, every layer's attention, acceptance, cache update
  draft       the draft side of one iteration: per tree level the draft layers' attention for the newest rows and the
              stop decision, which the host reads before it grows the next level
  verify      acceptance alone: one sequence to a serving batch, both tree modes, both sampling schemes, any vocabulary
  stop_rows   the early-stop model on draft distributions
  stop_hidden the early-stop model on draft hidden states

Shapes are those of the `workloads` package (Llama-2-7B's attention shape, vocabulary 32000, the paper's trees) and
neighbours of them.  q, k, v ~ N(0, 1); target logits ~ N(0, 3^2), draft logits = target + noise; tree tokens drawn from
the draft rows (level 1 of a target-initialised tree from the target row); uniforms in [0, 1).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2409_10644_amd import binding

BETA = 0.4                   # stop threshold
K_SCALE, V_SCALE = 0.05, 0.04   # scales of the fp8 cache: N(0, 1) values use most of the format's range
MAX_KV_BYTES, MAX_ATTN_FLOPS, MAX_F32_FLOPS, MAX_ROW_BYTES = 2.1e9, 2.5e11, 3.0e9, 1.3e9   # what a drawn case may cost

TREES = ("4,2,2,1", "3,2,2,1,1,1,1,1", "4,2,2,2", "8,2,2,1,1", "16,1,1,1,1", "2,4,3,1,1", "2,2,2", "1,1,1,1")


def _attention(name, dtype, B, H_q, H_kv, d, lo, hi, tree, gamma=0, newest=False):
    return {"name": name, "kind": "attention", "dtype": dtype, "B": B, "H_q": H_q, "H_kv": H_kv, "d": d, "prefix_min": lo,
            "prefix_max": hi, "tree": tree, "gamma": gamma or len(tree.split(",")), "newest": newest}


def listed():
    return [
        # the smallest call: a few heads of a small fp32 model, a short prompt; latency and launches
        _attention("f32_tiny", "f32", 1, 4, 4, 64, 128, 128, "2,2,2"),
        # one chat: 32 layers of a 7B model over 1024 cached tokens, (4,2,2,1) tree, acceptance and cache update
        {"name": "step_single", "kind": "step", "layers": 32, "B": 1, "H_q": 32, "d": 128, "prefix": 1024, "tree": "4,2,2,1", "V": 32000,
         "noise": 1.0},
        # the same user's draft side in the dynamic setting: width 16, depth 5, a two-layer draft model
        {"name": "draft_fork", "kind": "draft", "layers": 2, "B": 1, "H_q": 12, "d": 64, "prefix": 1024, "width": 16, "depth": 5, "V": 32000,
         "k": 10, "hidden": 64},
        # a serving batch: 16 conversations of very different lengths
        _attention("ragged_batch", "bf16", 16, 32, 32, 128, 512, 4096, "4,2,2,2"),
        # the largest call: long documents under the widest tree
        _attention("long_wide", "bf16", 8, 32, 32, 128, 16384, 16384, "8,2,2,1,1"),
        # the ragged batch on a model with grouped-query heads
        _attention("ragged_gqa", "bf16", 16, 32, 8, 128, 512, 4096, "4,2,2,2"),
        # the ragged batch with the cache quantised to 8 bits
        _attention("ragged_fp8", "fp8kv", 16, 32, 32, 128, 512, 4096, "4,2,2,2"),
        # acceptance for a serving batch, one tree each
        {"name": "verify_batch", "kind": "verify", "B": 128, "V": 32000, "tree": "4,2,2,1", "mode": "draft", "replacement": True, "n_new": 1,
         "noise": 1.0},
        # acceptance in target-initialised mode: eight walks per sequence, poor draft, next tree's first level drawn
        {"name": "verify_target", "kind": "verify", "B": 8, "V": 32000, "tree": "8,2,2,1,1", "mode": "target", "replacement": True, "n_new": 8,
         "noise": 2.0},
        # acceptance with a large vocabulary, siblings drawn without replacement
        {"name": "verify_large_vocab", "kind": "verify", "B": 16, "V": 131072, "tree": "4,2,2,2", "mode": "draft", "replacement": False,
         "n_new": 1, "noise": 1.5},
        # stop decisions of a large batch on the draft model's distributions
        {"name": "stop_rows_batch", "kind": "stop_rows", "B": 256, "W": 16, "V": 32000, "k": 10, "hidden": 64},
        # stop decisions on hidden states of a 768-wide draft model, three-layer network
        {"name": "stop_hidden_batch", "kind": "stop_hidden", "B": 64, "W": 16, "width": 768, "hidden1": 256, "hidden2": 64},
    ]


# ---------------------------------------------------------------------------------------------------- more cases
def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _vocab(rng):
    v = _log_int(rng, 4000, 262144)
    return v if rng.random() < 0.3 else v // 64 * 64         # vocabularies are mostly padded, not always


def _draw_attention(rng):
    dtype = rng.choice(("bf16", "bf16", "bf16", "fp8kv", "f32"))
    while True:
        tree = rng.choice(TREES)
        depth = len(tree.split(","))
        gamma = depth if rng.random() < 0.6 else rng.randint(1, depth)
        d = 128 if dtype == "fp8kv" or rng.random() < 0.75 else 64
        H_kv = rng.choice((4, 8, 12, 16, 32))
        grp = 1 if dtype == "f32" or rng.random() < 0.6 else rng.choice((2, 4, 8))
        hi = _log_int(rng, 64, 2048 if dtype == "f32" else 32768)
        lo = hi if rng.random() < 0.4 else max(1, hi // rng.choice((2, 4, 8)))
        c = _attention("", dtype, _log_int(rng, 1, 64), H_kv * grp, H_kv, d, lo, hi, tree, gamma, rng.random() < 0.2)
        if c["H_q"] > 64 or c["B"] * H_kv * hi * d * 4 > MAX_KV_BYTES:
            continue
        if work(c)["flops"] <= (MAX_F32_FLOPS if dtype == "f32" else MAX_ATTN_FLOPS):
            return c


def _draw_verify(rng):
    while True:
        tree = rng.choice(TREES)
        c = {"kind": "verify", "B": _log_int(rng, 1, 256), "V": _vocab(rng), "tree": tree, "mode": rng.choice(("draft", "draft", "target")),
             "replacement": rng.random() < 0.6, "n_new": 1, "noise": rng.choice((0.5, 1.0, 1.5, 2.0))}
        if c["mode"] == "target":
            c["n_new"] = int(tree.split(",")[0])
        n = _nodes(tree)
        if c["B"] * (n + 1) * c["V"] * 8 <= MAX_ROW_BYTES and c["B"] * c["n_new"] * c["V"] <= 128 * 65536:
            return c


def draw(rng):
    """One more case of the ranges above."""
    kind = rng.choice(("attention",) * 5 + ("step", "draft") + ("verify",) * 3 + ("stop_rows", "stop_hidden"))
    if kind == "attention":
        c = _draw_attention(rng)
    elif kind == "verify":
        c = _draw_verify(rng)
    elif kind == "step":
        B = rng.choice((1, 1, 1, 2, 4))
        c = {"kind": "step", "layers": rng.choice((16, 24, 32)), "B": B, "H_q": rng.choice((16, 32)), "d": 128,
             "prefix": _log_int(rng, 128, 2048 // B), "tree": rng.choice(TREES), "V": min(_vocab(rng), 65536), "noise": rng.choice((1.0, 1.5))}
    elif kind == "draft":
        c = {"kind": "draft", "layers": rng.choice((1, 2, 4)), "B": rng.choice((1, 1, 2, 4)), "H_q": rng.choice((8, 12, 16)), "d": 64,
             "prefix": _log_int(rng, 64, 4096), "width": rng.randint(4, 21), "depth": rng.randint(3, 6), "V": min(_vocab(rng), 65536),
             "k": rng.randint(4, 16), "hidden": rng.choice((32, 64, 128))}
    elif kind == "stop_rows":
        V, W = _vocab(rng), rng.randint(4, 21)
        c = {"kind": "stop_rows", "B": max(1, min(_log_int(rng, 1, 256), int(5e8 / (4 * V * W)))), "W": W, "V": V, "k": rng.randint(1, 16),
             "hidden": rng.choice((32, 64, 128))}
    else:
        c = {"kind": "stop_hidden", "B": _log_int(rng, 1, 64), "W": rng.randint(4, 21), "width": rng.choice((288, 512, 768, 1000, 1024, 2048)),
             "hidden1": rng.choice((64, 128, 256)), "hidden2": rng.choice((32, 64))}
    c.pop("name", None)
    return c


# ---------------------------------------------------------------------------------------------------- inputs
def _branching(tree):
    return [int(x) for x in tree.split(",")]


def _nodes(tree, gamma=None):
    n, total = 1, 0
    for b in _branching(tree)[:gamma]:
        n *= b
        total += n
    return total


def _rng(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, shape, dtype=torch.float32):
    return torch.randn(shape, generator=g, device="cuda", dtype=dtype)


def _prefix_lens(case, seed):
    r = np.random.Generator(np.random.PCG64(seed))
    lens = r.integers(case["prefix_min"], case["prefix_max"] + 1, size=case["B"]).astype(np.int32)
    lens[0] = case["prefix_max"]                     # the bound a caller passes is the longest length it has
    return r.permutation(lens)


def _prepare_attention(case, seed):
    g = _rng(seed)
    B, Hq, Hkv, d = case["B"], case["H_q"], case["H_kv"], case["d"]
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    n_max, gamma, mp = _nodes(case["tree"]), case["gamma"], case["prefix_max"]
    mask = binding.build_mask(_branching(case["tree"]))
    view = binding.slice_mask(mask, gamma)
    n = view.n_nodes
    row0 = view.level_off_host[gamma - 1] if case["newest"] else 0
    q = _normal(g, (B, Hq, n_max, d), dt)
    kt, vt = _normal(g, (B, Hkv, n_max, d), dt), _normal(g, (B, Hkv, n_max, d), dt)
    cap = mp + len(_branching(case["tree"]))         # room for one accepted path
    if case["dtype"] == "fp8kv":
        kp, vp = ((_normal(g, (B, Hkv, cap, d), torch.bfloat16) / s).to(torch.float8_e4m3fn).view(torch.uint8) for s in (K_SCALE, V_SCALE))
    else:
        kp, vp = _normal(g, (B, Hkv, cap, d), dt), _normal(g, (B, Hkv, cap, d), dt)
    lens = torch.from_numpy(_prefix_lens(case, seed)).cuda()
    base = torch.arange(B, dtype=torch.int64, device="cuda") * (Hkv * cap * d)
    out = torch.zeros_like(q)
    scale = 1.0 / math.sqrt(d)
    if case["dtype"] == "fp8kv":
        ws = binding.new_workspace(binding.tree_attention_fp8kv_workspace(B, Hq, Hkv, n, row0, mp))
        call = binding.tree_attention_fp8kv
        args = (view, B, Hq, Hkv, row0, q, kt, vt, n_max, kp, vp, K_SCALE, V_SCALE, base, lens, cap * d, mp, scale, out, ws)
    else:
        code = binding.MCSD_F32 if case["dtype"] == "f32" else binding.MCSD_BF16
        ws = binding.new_workspace(binding.tree_attention_gqa_workspace(B, Hq, Hkv, d, n, row0, mp))
        if Hq != Hkv:
            call, args = binding.tree_attention_gqa, (view, code, B, Hq, Hkv, d, row0, q)
        elif row0:
            call, args = binding.tree_attention_rows, (view, code, B, Hq, d, row0, q)
        else:
            call, args = binding.tree_attention, (view, code, B, Hq, d, q)
        args += (kt, vt, n_max, kp, vp, base, lens, cap * d, mp, scale, out, ws)
    return {"kind": "attention", "call": call, "args": args, "out": out}


def _run_attention(s):
    s["call"](*s["args"])
    return s["out"]


def _probabilities(g, B, V, tree, noise, mode, replacement, gamma):
    """Target rows, draft rows, tree tokens and uniforms of one verification."""
    br = _branching(tree)[:gamma]
    n, n_in = _nodes(tree, gamma), _nodes(tree, gamma - 1)
    logits = _normal(g, (B, 1 + n, V)).mul_(3.0)
    q = torch.softmax(logits[:, : 1 + n_in] + _normal(g, (B, 1 + n_in, V)).mul_(noise), dim=-1)
    p = torch.softmax(logits, dim=-1)
    tokens, first, parents = [], 0, 1                # contexts of a level: rows first .. first + parents - 1
    for level, b in enumerate(br):
        rows = p[:, :1] if mode == "target" and level == 0 else q[:, first:first + parents]
        x = torch.multinomial(rows.reshape(-1, V), b, replacement=replacement, generator=g)
        tokens.append(x.reshape(B, parents * b))
        first, parents = first + parents, parents * b
    tokens = torch.cat(tokens, dim=1).to(torch.int32).contiguous()
    ua = torch.rand((B, n), generator=g, device="cuda")
    return p, q, tokens, ua


def _prepare_verify(case, seed):
    g = _rng(seed)
    B, V, gamma = case["B"], case["V"], len(_branching(case["tree"]))
    mask = binding.build_mask(_branching(case["tree"]))
    view = binding.slice_mask(mask, gamma)
    p, q, tokens, ua = _probabilities(g, B, V, case["tree"], case["noise"], case["mode"], case["replacement"], gamma)
    n_new = case["n_new"]
    us = torch.rand((B, n_new), generator=g, device="cuda")
    mode = binding.MCSD_TARGET_INIT if case["mode"] == "target" else binding.MCSD_DRAFT_INIT
    path, alen, new = (torch.zeros(shape, dtype=torch.int32, device="cuda") for shape in ((B, gamma), (B,), (B, n_new)))
    ws_bytes = binding.verify_tree_workspace(view, mode, B, n_new)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda") if ws_bytes else None
    tail = (B, V, tokens, p, q, p.stride(0), q.stride(0), ua, us, n_new, path, alen, new, ws)
    if case["replacement"]:
        call, args = binding.verify_tree, (view, mode) + tail
    else:
        call, args = binding.verify_tree_sampling, (view, mode, binding.MCSD_WITHOUT_REPLACEMENT) + tail
    return {"kind": "verify", "call": call, "args": args, "out": (path, alen, new)}


def _prepare_step(case, seed):
    g = _rng(seed)
    n_layers, B, H, d, L, V, tree = (case[x] for x in ("layers", "B", "H_q", "d", "prefix", "V", "tree"))
    n, gamma = _nodes(tree), len(_branching(tree))
    cap = L + gamma
    bf16 = torch.bfloat16
    q, kt, vt = (_normal(g, (n_layers, B, H, n, d), bf16) for _ in range(3))
    kp, vp = (_normal(g, (n_layers, B, H, cap, d), bf16) for _ in range(2))
    out = torch.zeros_like(q)
    p, dq, tokens, ua = _probabilities(g, B, V, tree, case["noise"], "draft", True, gamma)
    i32 = dict(dtype=torch.int32, device="cuda")
    s = {"kind": "step", "case": case, "mask": binding.build_mask(_branching(tree)), "gamma": gamma, "n": n, "cap": cap,
         "layers": [tuple(x[l] for x in (q, kt, vt, kp, vp, out)) for l in range(n_layers)], "p": p, "dq": dq, "tokens": tokens,
         "ua": ua, "us": torch.rand((B, 1), generator=g, device="cuda"), "kp": kp, "vp": vp, "out": out,
         "base": torch.arange(B, dtype=torch.int64, device="cuda") * (H * cap * d), "lens": torch.full((B,), L, **i32),
         "path": torch.zeros((B, gamma), **i32), "alen": torch.zeros((B,), **i32), "new": torch.zeros((B, 1), **i32),
         "ids": torch.zeros((B, gamma + 1), **i32), "n_ids": torch.zeros((B,), **i32),
         "ws": binding.new_workspace(binding.tree_attention_workspace(B, H, d, n, L)), "scale": 1.0 / math.sqrt(d)}
    s["tree_k"], s["tree_v"], s["cache_k"], s["cache_v"] = ([layer[i] for layer in s["layers"]] for i in (1, 2, 3, 4))
    return s


def _run_step(s):
    # The prefix bound stays at the state's length, so a length that an earlier pass advanced counts as that length
    # again and every pass is the same step.
    c = s["case"]
    B, H, d, L, V = c["B"], c["H_q"], c["d"], c["prefix"], c["V"]
    n, cap, lens, base = s["n"], s["cap"], s["lens"], s["base"]
    view = binding.slice_mask(s["mask"], s["gamma"])
    for q, kt, vt, kp, vp, out in s["layers"]:
        binding.tree_attention(view, binding.MCSD_BF16, B, H, d, q, kt, vt, n, kp, vp, base, lens, cap * d, L, s["scale"], out, s["ws"])
    p, dq = s["p"], s["dq"]
    binding.verify_tree(view, binding.MCSD_DRAFT_INIT, B, V, s["tokens"], p, dq, p.stride(0), dq.stride(0), s["ua"], s["us"], 1,
                        s["path"], s["alen"], s["new"], None)
    binding.commit_path(view, binding.MCSD_BF16, B, H, d, s["tree_k"], s["tree_v"], n, s["cache_k"], s["cache_v"], base, cap * d, L, cap,
                        s["path"], s["alen"], s["tokens"], s["new"], 1, 1, lens, s["ids"], s["n_ids"])
    return {x: s[x] for x in ("out", "kp", "vp", "path", "alen", "new", "ids", "n_ids", "lens")}


def _mlp(g, widths, out_bias=0.0):
    ws = [_normal(g, (o, i)) * math.sqrt(2.0 / i) for i, o in zip(widths[:-1], widths[1:])]
    bs = [_normal(g, (o,)) * 0.1 for o in widths[1:]]
    bs[-1] += out_bias
    return binding.make_mlp(ws, bs)


def _draft_rows(g, B, rows, V, noise=1.0):
    return torch.softmax(_normal(g, (B, rows, V)).mul_(3.0) + _normal(g, (B, rows, V)).mul_(noise), dim=-1)


def _prepare_draft(case, seed):
    g = _rng(seed)
    n_layers, B, H, d, L, W, D, V = (case[x] for x in ("layers", "B", "H_q", "d", "prefix", "width", "depth", "V"))
    n, cap, bf16 = W * D, L + D, torch.bfloat16
    q, kt, vt = (_normal(g, (n_layers, B, H, n, d), bf16) for _ in range(3))
    kp, vp = (_normal(g, (n_layers, B, H, cap, d), bf16) for _ in range(2))
    out = torch.zeros_like(q)
    rows = _draft_rows(g, B, n - W, V)               # the draft distributions after the nodes of levels 1 .. D-1
    ws = max(binding.tree_attention_rows_workspace(B, H, d, W * l, W * (l - 1), L) for l in range(1, D + 1))
    return {"kind": "draft", "case": case, "mask": binding.build_mask([W] + [1] * (D - 1)), "cap": cap, "rows": rows,
            "layers": [tuple(x[l] for x in (q, kt, vt, kp, vp, out)) for l in range(n_layers)], "out": out,
            "base": torch.arange(B, dtype=torch.int64, device="cuda") * (H * cap * d), "n": n,
            "lens": torch.full((B,), L, dtype=torch.int32, device="cuda"), "ws": binding.new_workspace(ws), "scale": 1.0 / math.sqrt(d),
            # a model that lets the tree grow to its full depth
            "mlp": _mlp(g, (case["k"] + 1, case["hidden"], 1), out_bias=12.0),
            "prob": torch.zeros((D - 1, B, W), device="cuda"), "stop": torch.zeros((D - 1, B), dtype=torch.int32, device="cuda"),
            "stop_host": torch.zeros((B,), dtype=torch.int32, pin_memory=True)}


def _run_draft(s):
    c = s["case"]
    B, H, d, L, W, V = c["B"], c["H_q"], c["d"], c["prefix"], c["width"], c["V"]
    n, cap, rows, stop_host = s["n"], s["cap"], s["rows"], s["stop_host"]
    for level in range(1, c["depth"] + 1):
        view = binding.slice_mask(s["mask"], level)
        first = W * (level - 1)
        for q, kt, vt, kp, vp, out in s["layers"]:
            binding.tree_attention_rows(view, binding.MCSD_BF16, B, H, d, first, q, kt, vt, n, kp, vp, s["base"], s["lens"], cap * d, L,
                                        s["scale"], out, s["ws"])
        if level == c["depth"]:
            break
        stop = s["stop"][level - 1]
        binding.early_stop_distribution(s["mlp"], B, W, V, c["k"], rows[:, first:], rows.stride(0), V, BETA, None, s["prob"][level - 1], stop)
        stop_host.copy_(stop, non_blocking=True)     # the loop waits for this decision
        torch.cuda.current_stream().synchronize()
        if bool(stop_host.all()):
            break
    return s["out"], s["prob"], s["stop"]


def _prepare_stop(case, seed):
    g = _rng(seed)
    B, W = case["B"], case["W"]
    prob, stop = torch.zeros((B, W), device="cuda"), torch.zeros((B,), dtype=torch.int32, device="cuda")
    if case["kind"] == "stop_rows":
        V, k = case["V"], case["k"]
        rows = _draft_rows(g, B, W, V)
        features = torch.zeros((B, W, k + 1), device="cuda")
        mlp = _mlp(g, (k + 1, case["hidden"], 1))
        return {"kind": "stop", "call": binding.early_stop_distribution,
                "args": (mlp, B, W, V, k, rows, rows.stride(0), V, BETA, features, prob, stop), "out": (features, prob, stop)}
    width = case["width"]
    hidden = _normal(g, (B, W, width))
    mlp = _mlp(g, (width, case["hidden1"], case["hidden2"], 1))
    return {"kind": "stop", "call": binding.early_stop_hidden,
            "args": (mlp, B, W, hidden, W * width, width, BETA, prob, stop), "out": (prob, stop)}


_PREPARE = {"attention": _prepare_attention, "step": _prepare_step, "draft": _prepare_draft, "verify": _prepare_verify,
            "stop_rows": _prepare_stop, "stop_hidden": _prepare_stop}


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, seed)


def run(state):
    kind = state["kind"]
    if kind == "step":
        return _run_step(state)
    if kind == "draft":
        return _run_draft(state)
    if kind == "attention":
        return _run_attention(state)
    state["call"](*state["args"])
    return state["out"]


# ---------------------------------------------------------------------------------------------------- what a pass needs
def _attention_work(dtype, B, H_q, H_kv, d, L, n, rows):
    e = 4 if dtype == "f32" else 2
    cache = 2 * B * H_kv * L * d * (1 if dtype == "fp8kv" else e)
    tree = 2 * B * H_kv * n * d * e
    return cache + tree + 2 * B * H_q * rows * d * e, 4.0 * B * H_q * rows * (L + n) * d


def _mlp_work(rows, widths):
    weights = sum(i * o + o for i, o in zip(widths[:-1], widths[1:]))
    return 4 * weights, 2.0 * rows * weights


def work(case):
    kind, B = case["kind"], case["B"]
    if kind == "attention":
        n = _nodes(case["tree"], case["gamma"])
        rows = n - _nodes(case["tree"], case["gamma"] - 1) if case["newest"] else n
        L = (case["prefix_min"] + case["prefix_max"]) / 2
        by, fl = _attention_work(case["dtype"], B, case["H_q"], case["H_kv"], case["d"], L, n, rows)
    elif kind == "step":
        n = _nodes(case["tree"])
        by, fl = _attention_work("bf16", B, case["H_q"], case["H_q"], case["d"], case["prefix"], n, n)
        # acceptance: the two rows of the context at which the walk ends (or one row after the last node)
        by, fl = case["layers"] * by + B * 8 * case["V"], case["layers"] * fl + 3.0 * B * case["V"]
    elif kind == "draft":
        W, D, by, fl = case["width"], case["depth"], 0, 0.0
        for level in range(1, D + 1):
            b, f = _attention_work("bf16", B, case["H_q"], case["H_q"], case["d"], case["prefix"], W * level, W)
            by, fl = by + case["layers"] * b, fl + case["layers"] * f
        by, fl = by + 4 * B * W * (D - 1) * case["V"], fl + 3.0 * B * W * (D - 1) * case["V"]
    elif kind == "verify":
        walks = B * (_branching(case["tree"])[0] if case["mode"] == "target" else 1)
        by, fl = walks * 8 * case["V"], 3.0 * walks * case["V"]
    elif kind == "stop_rows":
        m = B * case["W"]
        b, f = _mlp_work(m, (case["k"] + 1, case["hidden"], 1))
        by, fl = b + 4 * m * (case["V"] + case["k"] + 2), f + 3.0 * m * case["V"]
    else:
        m = B * case["W"]
        b, f = _mlp_work(m, (case["width"], case["hidden1"], case["hidden2"], 1))
        by, fl = b + 4 * m * (case["width"] + 1), f
    return {"bytes": by, "flops": fl}


def tolerance(case):
    kind = case["kind"]
    if kind == "verify":
        return "exact"                               # paths, lengths and tokens are specified bit for bit
    if kind == "stop_rows" or kind == "stop_hidden":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.005}      # fp32; a probability at the threshold may fall either way
    if kind == "attention" and case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.08}                # bf16 scores' exponentials, partial sums and outputs; ids are exact
