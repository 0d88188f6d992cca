#!/usr/bin/env python3
"""Benchmark of the MCSD verification hot path on one MI355X.

One STEP is one pass of the whole hot path over one batch of seeded synthetic input:
    mcsd_slice_mask(gamma)  ->  one mcsd_tree_attention call per transformer layer (32 for Llama-2-7B, every
    layer with its own KV cache and q/k/v)  ->  one mcsd_verify_tree call.
All inputs are resident in HBM before the timed region.  The headline value is verified tree-tokens/s =
B * N(gamma) / step time on cfg2 (the configuration the metric is quoted on).  The line also carries the roofline of
the dominant kernel (the tree-attention key sweep), measured with HIP events that bracket that kernel's launches, the
CPU oracle timed on the host cores as a reported baseline, and one section per other configuration.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload cfg2] [--extra cfg1,cfg3,cfg4,cfg5,cfg4_b64]
"""
from __future__ import annotations

import argparse
import json
import os
import re
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)
sys.path.insert(0, os.path.join(ROOT, "tests"))

HBM_PEAK_GBPS = 8000.0          # MI355X HBM3E, published
MFMA_BF16_PEAK_TFLOPS = 2500.0  # dense bf16, published
N_LAYERS = 32                   # Llama-2-7B
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "tree_attn_hbm_traffic_pmc.md")


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def measured_traffic():
    """HBM bytes per launch of the sweep kernel from the rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs summarised in
    profiles/: rows `| workload | kernel instantiation | workgroups | fetched bytes | written bytes |`, keyed by
    (instantiation, grid).  A launch whose key is not in the file has no measured traffic (null in the output)."""
    table = {}
    try:
        with open(TRAFFIC_FILE) as f:
            for line in f:
                m = re.match(r"^\|[^|]*\|\s*`?(tree_attn_\w+<[^>|]*>)`?\s*\|\s*(\d+)\s*\|\s*([\d ]+)\|\s*([\d ]+)\|", line)
                if m:
                    table[(m.group(1).replace(" ", ""), int(m.group(2)))] = \
                        int(m.group(3).replace(" ", "")) + int(m.group(4).replace(" ", ""))
    except OSError:
        pass
    return table


def attention_algorithmic(w, lens, n, kv_bytes_per_elem=None):
    """Algorithmic bytes and flops of one mcsd_tree_attention call: prefix K and V read once, tree q/k/v read and
    the output written once, plus the mask slice; 4*N*(L+N)*d flops per (sequence, head)."""
    e = 2 if w.dtype == "bf16" else 4
    ekv = e if kv_bytes_per_elem is None else kv_bytes_per_elem
    by = sum(w.H * w.d * (2 * int(L) * ekv + 4 * n * e) for L in lens) + n * ((w.n_nodes() + 63) // 64) * 8
    fl = sum(w.H * 4 * n * (int(L) + n) * w.d for L in lens)
    return by, fl


def walk_bytes(w, gamma, mode, n_new, paths, lens):
    """Vocabulary bytes the acceptance walks have to read, from their own results.  paths / lens: one entry per walk
    (draft-initialised: one per sequence from the context that ends the prefix; target-initialised: one per level-1
    node, whose first entry is that node, accepted untested).  A context with at least one rejection needs its target
    and draft row (2 * V * 4 bytes, read once); a walk that accepts at every level needs the target row after its last
    node for the new tokens (V * 4 bytes; after a rejection the new tokens come from the residual the walk already
    holds); every tested candidate needs p(x), q(x), its token id and its uniform (16 bytes)."""
    br = list(w.branching[:gamma])
    off = [0]
    for l, b in enumerate(br):
        off.append(off[-1] + (b if l == 0 else (off[-1] - off[-2]) * b))
    total = 0
    for path, ln in zip(paths, lens):
        cur, level = -1, 0
        if mode == 1:
            cur, level = int(path[0]), 1
        while level < gamma:
            cnt = br[level]
            first = 0 if cur < 0 else off[level] + (cur - off[level - 1]) * cnt
            if level < ln:
                rejected = int(path[level]) - first
                total += 16 * (rejected + 1) + (2 * w.V * 4 if rejected else 0)
                cur = int(path[level])
                level += 1
            else:
                total += 16 * cnt + 2 * w.V * 4          # every child rejected: the walk ends here
                break
        else:
            total += w.V * 4 if n_new else 0             # all levels accepted
    return total


class Step:
    """Device-resident inputs of one step and the calls that make it."""

    def __init__(self, name, n_kv_sets, gamma=None, mode=None, seed=0, verify_seed=None, tuning=None):
        import numpy as np
        import torch
        from paper_2409_10644_amd import binding
        from workloads import WORKLOADS, attention_inputs, prefix_lens
        import gpu_helpers as H

        self.binding, self.H, self.torch, self.np = binding, H, torch, np
        self.w = w = WORKLOADS[name]
        self.gamma = w.gamma_max if gamma is None else gamma
        self.mode = w.mode if mode is None else mode
        self.lens = prefix_lens(w, seed)
        self.cap = int(w.prefix_max)
        t0 = time.time()
        self.layers_host = [attention_inputs(w, seed=seed, kv_capacity=self.cap, variant=l) for l in range(n_kv_sets)]
        self.layers = [H.AttnDevice(inp) for inp in self.layers_host]
        log(f"[bench] {name}: {n_kv_sets} KV set(s) generated and uploaded in {time.time() - t0:.1f}s")
        self.mask = binding.build_mask(w.branching)                   # once, at gamma_max
        self.tuning = tuning                                          # None: the library's own plan
        self.set_gamma(self.gamma)
        self.set_verify_inputs(seed if verify_seed is None else verify_seed)

    def set_gamma(self, gamma):
        b, w = self.binding, self.w
        self.gamma = gamma
        self.view = b.slice_mask(self.mask, gamma)
        self.n = self.view.n_nodes
        self.ws_bytes = b.tree_attention_tuned_workspace(self.tuning, 0, w.B, w.H, w.H, w.d, self.n, 0, self.cap)
        self.ws = b.new_workspace(self.ws_bytes)
        self.plan = b.tree_attention_plan(self.tuning, 1 if w.dtype == "bf16" else 0, 0, w.B, w.H, w.H, w.d, self.n, 0, self.cap)
        self.alg_bytes, self.alg_flops = attention_algorithmic(w, self.lens, self.n)

    def set_verify_inputs(self, seed, vi=None):
        from workloads import verify_inputs
        torch, H, w, b = self.torch, self.H, self.w, self.binding
        self.vi = vi = verify_inputs(w, seed=seed, gamma=self.gamma, mode=self.mode) if vi is None else vi
        self.p, self.q = H.dev(vi["p_target"]), H.dev(vi["q_draft"])
        self.tokens, self.ua, self.us = H.dev(vi["tokens"]), H.dev(vi["u_accept"]), H.dev(vi["u_sample"])
        self.n_new = vi["n_new"]
        self.path = torch.zeros((w.B, self.gamma), dtype=torch.int32, device="cuda")
        self.alen = torch.zeros((w.B,), dtype=torch.int32, device="cuda")
        self.new = torch.zeros((w.B, max(self.n_new, 1)), dtype=torch.int32, device="cuda")
        vws = b.verify_tree_workspace(self.view, self.mode, w.B, self.n_new)
        self.vws = torch.zeros(max(vws, 256), dtype=torch.uint8, device="cuda") if vws else None

    def kernel_name(self):
        if not self.plan.mfma_path:
            return f"tree_attn_f32_kernel<{self.w.d}>"
        keys = 128 if self.plan.query_blocks == 1 else 64       # of a tile; split prefixes below 512 keys exchange fp32
        short = "_short" if self.plan.key_splits > 1 and -(-self.cap // keys) * keys < 512 else ""
        pairs = self.plan.ordered_by_length and self.plan.key_splits == 1 and self.plan.workgroups <= 512    # long and short ones, two per compute unit
        ragged = "_ragged" if pairs and self.plan.query_blocks != 4 and (self.w.d, self.plan.query_blocks) != (128, 1) else ""
        return f"tree_attn_bf16{short}{ragged}_kernel<{self.w.d}, {self.plan.query_blocks}, {self.plan.stages}, false>"

    def attention(self, layer):
        ad, w, b = self.layers[layer % len(self.layers)], self.w, self.binding
        if self.tuning is None:
            b.tree_attention(self.view, ad.code, w.B, w.H, w.d, ad.q, ad.kt, ad.vt, ad.node_stride, ad.kp, ad.vp, ad.base,
                             ad.lens, ad.head_stride, self.cap, ad.scale, ad.out, self.ws)
        else:
            b.tree_attention_tuned(self.tuning, self.view, ad.code, 0, 1.0, 1.0, w.B, w.H, w.H, w.d, 0, ad.q, ad.kt, ad.vt,
                                   ad.node_stride, ad.kp, ad.vp, ad.base, ad.lens, ad.head_stride, self.cap, ad.scale,
                                   ad.out, self.ws)

    def verify(self):
        w, b, vi = self.w, self.binding, self.vi
        b.verify_tree(self.view, self.mode, w.B, w.V, self.tokens, self.p, self.q, vi["p_target"].shape[1] * w.V,
                      vi["q_draft"].shape[1] * w.V, self.ua, self.us, self.n_new, self.path, self.alen, self.new,
                      self.vws)

    def commit(self, lens_dev, ids, n_ids):
        """Update after acceptance over all layers' caches (not part of the timed step: the row after it).  The
        benchmark's caches are exactly prefix_max rows long, so lengths are clamped gamma rows below that."""
        w, b = self.w, self.binding
        L = self.layers
        b.commit_path(self.view, L[0].code, w.B, w.H, w.d, [a.kt for a in L], [a.vt for a in L], L[0].node_stride,
                      [a.kp for a in L], [a.vp for a in L], L[0].base, L[0].head_stride, self.cap - self.gamma, self.cap,
                      self.path, self.alen, self.tokens, self.new, self.n_new, 1 if self.mode == 0 else 0, lens_dev,
                      ids, n_ids)

    def step(self):
        self.view = self.binding.slice_mask(self.mask, self.gamma)    # O(1): the per-step slice
        for l in range(N_LAYERS):
            self.attention(l)
        self.verify()

    def walks(self):
        """(paths, lengths) of all walks of the last verify call, as numpy (see walk_bytes)."""
        np_, w = self.np, self.w
        if self.mode == 0:
            return self.path.cpu().numpy(), self.alen.cpu().numpy()
        R, g = int(w.branching[0]), self.gamma               # the workspace keeps every level-1 subtree's walk
        raw = self.vws.cpu().numpy()
        a256 = lambda x: (x + 255) & ~255
        paths = raw[:4 * w.B * R * g].view(np_.int32).reshape(w.B * R, g)
        o = a256(4 * w.B * R * g)
        lens = raw[o:o + 4 * w.B * R].view(np_.int32).reshape(w.B * R)
        return paths, lens

    def check_against_oracle(self):
        """'Verified': the outputs of this very configuration match the oracle: EVERY element of layer 0's attention
        output (the buffer starts as NaN) and the full verification result.  Returns (mean accepted length, seconds
        the oracle took for the attention layer)."""
        import oracle
        np_, torch = self.np, self.torch
        w = self.w
        self.layers[0].out.fill_(float("nan"))
        self.attention(0)
        self.verify()
        torch.cuda.synchronize()
        M = oracle.build_mask(w.branching)
        got = self.layers[0].out[:, :, :self.n].float().cpu().numpy().astype(np_.float64)
        t0 = time.time()
        want = oracle.tree_attention(self.layers_host[0], M, self.n)
        t_attn = time.time() - t0
        self.H.assert_close(got, want, w.dtype, f"bench {w.name} gamma={self.gamma}, every element")
        vi = self.vi
        want_v = oracle.verify_tree(self.mode, w.branching[:self.gamma], vi["tokens"], vi["p_target"], vi["q_draft"],
                                    vi["u_accept"], vi["u_sample"])
        got_v = (self.path.cpu().numpy(), self.alen.cpu().numpy(), self.new.cpu().numpy()[:, :self.n_new])
        for a, b_ in zip(got_v, want_v):
            assert np_.array_equal(a, b_), "verification differs from the oracle"
        return float(want_v[1].mean()), t_attn


class Ctx:
    """What time_kernel needs of a Step, for the sections that are not a Step."""

    def __init__(self, binding, torch):
        self.binding, self.torch = binding, torch


def time_kernel(st, hip, kernel_id, launch, reps, warm=0):
    """Average device execution time (ms) of one library kernel over `reps` back-to-back launches, from event
    pairs that the library places around that kernel's launch.  `warm` untimed launches go first in the same
    burst, so that the timed ones see the clocks of sustained work rather than the ramp out of idle."""
    b, torch = st.binding, st.torch
    pairs = [(hip.event(), hip.event()) for _ in range(reps)]
    for i in range(warm):
        launch(i)
    for i, (e0, e1) in enumerate(pairs):
        b.profile_next(kernel_id, e0, e1)
        launch(warm + i)
    torch.cuda.synchronize()
    ms = [hip.elapsed_ms(e0, e1) for e0, e1 in pairs]
    for e0, e1 in pairs:
        hip.destroy(e0)
        hip.destroy(e1)
    ms.sort()
    return sum(ms) / len(ms), ms[len(ms) // 2], ms[len(ms) // 10], ms[(len(ms) * 9) // 10]


def time_in_graph(st, hip, launch, per_graph, replays):
    """Average duration (ms) of one launch inside a HIP graph of `per_graph` back-to-back launches, from one pair of HIP
    events on the stream around `replays` replays (after as many untimed ones).  For kernels of a few microseconds: an
    event pair around a single launch adds ~1 us of dispatch time, back-to-back launches show what a launch costs in
    the step (the kernel trace of the replayed step agrees with this figure)."""
    torch = st.torch
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for i in range(per_graph):
            launch(i)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for i in range(per_graph):
            launch(i)
    for _ in range(replays):
        g.replay()
    e0, e1 = hip.event(), hip.event()
    hip.record(e0)
    for _ in range(replays):
        g.replay()
    hip.record(e1)
    ms = hip.elapsed_ms(e0, e1)
    hip.destroy(e0)
    hip.destroy(e1)
    del g
    return ms / (replays * per_graph)


def roofline_of(st, hip, reps, traffic, warm=0):
    b = st.binding
    avg, med, p10, p90 = time_kernel(st, hip, b.KERNEL_ATTN_SWEEP, lambda i: st.attention(i), reps, warm)
    pair_avg = None
    if st.alg_bytes < 1e8 and (st.plan.fold_in_kernel or st.plan.key_splits == 1):
        # a launch of a few microseconds that is one kernel: timed back to back inside a graph (see time_in_graph)
        try:
            pair_avg, avg = avg, time_in_graph(st, hip, lambda i: st.attention(i), N_LAYERS, 20)
        except Exception as ex:
            log(f"[bench] in-graph timing failed ({ex!r}); keeping the event pairs")
            pair_avg = None
    ach = st.alg_bytes / (avg * 1e-3) / 1e9
    kname = st.kernel_name()
    return {"bound": "hbm", "kernel": kname, "workgroups": int(st.plan.workgroups), "key_splits": int(st.plan.key_splits),
            "fold_in_kernel": bool(st.plan.fold_in_kernel),
            "achieved": round(ach, 1), "peak": HBM_PEAK_GBPS, "unit": "GB/s", "frac": round(ach / HBM_PEAK_GBPS, 4),
            "traffic": traffic.get((kname.replace(" ", ""), int(st.plan.workgroups))),
            "algorithmic_bytes_per_launch": int(st.alg_bytes),
            "flops_per_launch": int(st.alg_flops), "avg_launch_us": round(avg * 1e3, 2),
            "timed": ("one HIP event pair around 20 replays of a graph of %d back-to-back launches" % N_LAYERS) if pair_avg is not None
                     else "HIP event pair around every launch",
            "event_pair_launch_us": round((pair_avg if pair_avg is not None else avg) * 1e3, 2),
            "median_launch_us": round(med * 1e3, 2), "p10_us": round(p10 * 1e3, 2), "p90_us": round(p90 * 1e3, 2),
            "mfma_tflops": round(st.alg_flops / (avg * 1e-3) / 1e12, 1), "launches_timed": reps}


_FLUSH = None


def flush_caches(torch, i):
    """Overwrites 512 MB (twice the last-level cache), so that the next kernel finds none of its inputs in a cache."""
    global _FLUSH
    if _FLUSH is None:
        _FLUSH = torch.empty(512 << 20, dtype=torch.uint8, device="cuda")
    _FLUSH.fill_(i & 1)


def walk_kernel(V, walks):
    """The verification kernel of a launch: teams of workgroups, or one workgroup per walk where a vocabulary of up to 32768
    entries meets more walks than leave two compute units each."""
    return "verify_walk_fast_kernel" if V < 4 or (16384 < V <= 32768 and 2 * walks > 256) else "verify_walk_team_kernel"


def verify_section(st, hip, reps):
    """The verification call of a Step as it stands: kernel time, the vocabulary bytes its walks need, acceptance.
    The probability rows of one call (a few MB) would stay in the last-level cache between launches, so the figure
    set against the HBM peak is timed with the caches overwritten before every launch; the time with the rows still
    cached is reported beside it."""
    b, torch = st.binding, st.torch
    v_warm = time_kernel(st, hip, b.KERNEL_VERIFY_WALK, lambda i: st.verify(), reps, warm=8)[0]

    def cold(i):
        flush_caches(torch, i)
        st.verify()
    v_avg = time_kernel(st, hip, b.KERNEL_VERIFY_WALK, cold, min(reps, 24), warm=2)[0]
    torch.cuda.synchronize()
    paths, lens = st.walks()
    vb = walk_bytes(st.w, st.gamma, st.mode, st.n_new, paths, lens)
    alen = st.alen.cpu().numpy().astype(float)
    tested = st.gamma - (1 if st.mode else 0)
    return {"bound": "hbm", "kernel": walk_kernel(st.w.V, len(lens)),
            "mode": "target-init" if st.mode else "draft-init", "walks": int(len(lens)),
            "achieved": round(vb / (v_avg * 1e-3) / 1e9, 2), "peak": HBM_PEAK_GBPS, "unit": "GB/s",
            "frac": round(vb / (v_avg * 1e-3) / 1e9 / HBM_PEAK_GBPS, 5), "algorithmic_bytes_per_launch": int(vb),
            "avg_launch_us": round(v_avg * 1e3, 2), "rows_still_cached_launch_us": round(v_warm * 1e3, 2),
            "verify_tree_tokens_per_s": round(st.w.B * st.n / (v_avg * 1e-3), 1),
            "mean_accept_len": round(float(alen.mean()), 3),
            "alpha": round(float((alen.mean() - (1 if st.mode else 0)) / tested), 3) if tested > 0 else None}


def pick_verify_seed(w, gamma, mode, n_seeds=16):
    """The acceptance walk of one sequence depends on its draw; the timed step uses the seed (of 0..n_seeds-1) whose
    accepted length is closest to the mean over those seeds (lowest seed on ties), decided by the oracle.  Returns
    (seed, per-seed inputs, per-seed accepted lengths)."""
    import numpy as np
    import oracle
    from workloads import verify_inputs
    vis, lens = [], []
    for s in range(n_seeds):
        vi = verify_inputs(w, seed=s, gamma=gamma, mode=mode)
        want = oracle.verify_tree(mode, w.branching[:gamma], vi["tokens"], vi["p_target"], vi["q_draft"], vi["u_accept"],
                                  vi["u_sample"])
        vis.append(vi)
        lens.append(float(want[1].mean()))
    mean = float(np.mean(lens))
    seed = min(range(n_seeds), key=lambda s: (abs(lens[s] - mean), s))
    return seed, vis, lens


def timed_steps(st, torch, steps, warmup, eager, ramp_ms=25.0):
    """Captures the step into a HIP graph (unless eager), runs untimed steps until the chip has left its idle clocks
    (at least `warmup` steps and at least ramp_ms of back-to-back work), then times `steps` steps."""
    run_step, launch, graph = st.step, "eager", None
    if not eager:
        try:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                st.step()
            torch.cuda.current_stream().wait_stream(side)
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                st.step()
            run_step, launch = graph.replay, "hip-graph"
        except Exception as ex:
            log(f"[bench] graph capture failed ({ex!r}); timing eager launches")
    torch.cuda.synchronize()
    n_ramp, t0 = 0, time.perf_counter()
    while n_ramp < warmup or (time.perf_counter() - t0) * 1e3 < ramp_ms:
        run_step()
        n_ramp += 1
        if n_ramp % 8 == 0:
            torch.cuda.synchronize()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        run_step()
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    if launch == "hip-graph":                     # the replayed step must leave what the eager step leaves
        last = st.layers[(N_LAYERS - 1) % len(st.layers)].out
        got_v = (st.path.clone(), st.alen.clone(), st.new.clone(), last.clone())
        st.step()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got_v, (st.path, st.alen, st.new, last))), \
            "graph replay differs from eager launches"
    return dt / steps * 1e3, launch, n_ramp, graph


def cpu_baseline(st, t_attn_layer):
    """The oracle as it stands on the host cores: one attention layer in full (the run that checked the GPU's output)
    and one verification, scaled to a step of 32 layers; tree-tokens/s of a whole step."""
    import oracle
    w, vi = st.w, st.vi
    t0 = time.time()
    oracle.verify_tree(st.mode, w.branching[:st.gamma], vi["tokens"], vi["p_target"], vi["q_draft"], vi["u_accept"],
                       vi["u_sample"])
    t_verify = time.time() - t0
    t_step = N_LAYERS * t_attn_layer + t_verify
    return {"value": round(w.B * st.n / t_step, 3), "unit": "tree-tokens/s", "cores": oracle.threads(), "kind": "oracle",
            "sample": f"1 of {N_LAYERS} attention layers in full ({w.B * w.H * st.n} output rows) + 1 verification, "
                      f"attention time scaled to {N_LAYERS} layers",
            "attention_layer_s": round(t_attn_layer, 4), "verify_s": round(t_verify, 4)}


def config_section(name, hip, args, traffic, gammas=(None,), n_sets=1, with_step=False):
    """Attention roofline, verification and (optionally) the whole step of one of the other configurations, each
    checked against the oracle first.  One entry per gamma."""
    import torch
    out = {}
    es = Step(name, n_sets)
    for g in gammas:
        tag = name if g is None or g == es.w.gamma_max else f"{name}_gamma{g}"
        if g is not None:
            es.set_gamma(g)
            es.set_verify_inputs(0)
        alpha, t_attn = es.check_against_oracle()
        for i in range(3):
            es.attention(i)
        reps = args.extra_reps if es.alg_bytes > 1e8 else args.kernel_reps
        r = roofline_of(es, hip, reps, traffic, warm=reps)
        torch.cuda.synchronize()
        # The same launch out of a short idle period: the figures above are sustained ones (the chip lowers its clocks
        # under the combined load of the matrix cores and the memory stream); this one shows what that costs.
        time.sleep(0.05)
        r["launch_after_idle_us"] = round(time_kernel(es, hip, es.binding.KERNEL_ATTN_SWEEP, lambda i: es.attention(i), 3)[0] * 1e3, 2)
        t0e = time.perf_counter()
        for i in range(reps):
            es.attention(i)
        torch.cuda.synchronize()
        call_us = (time.perf_counter() - t0e) / reps * 1e6
        r["attention_call_us"] = round(call_us, 1)
        r["attn_tree_tokens_per_s"] = round(es.w.B * es.n / (call_us * 1e-6), 1)
        r["workload"] = (f"{name}: B{es.w.B} H{es.w.H} d{es.w.d} {es.w.dtype} N={es.n} gamma={es.gamma} "
                         f"prefix {es.w.prefix_min}-{es.w.prefix_max}")
        r["verified_vs_oracle"] = "every element of one layer's output + the verification result"
        r["verify"] = verify_section(es, hip, args.kernel_reps)
        r["step_tree_tokens_per_s_projected"] = round(
            es.w.B * es.n / (N_LAYERS * call_us * 1e-6 + r["verify"]["avg_launch_us"] * 1e-6), 1)
        if not args.no_cpu_baseline:
            r["cpu_baseline"] = cpu_baseline(es, t_attn)
        if with_step:
            ms, launch, n_ramp, graph = timed_steps(es, torch, args.steps, args.warmup, args.eager)
            r["step"] = {"ms_per_step": round(ms, 4), "tree_tokens_per_s": round(es.w.B * es.n / (ms * 1e-3), 1),
                         "launch": launch, "kv_sets": n_sets, "steps": args.steps}
            del graph
        out[tag] = r
    del es
    torch.cuda.empty_cache()
    return out


def dynamic_section(binding, torch, iterations):
    """One iteration of the dynamic setting (Sec. 3.2, 3.3; width 16, depth 5 of Sec. 4.1) on the fork-shaped tree:
    per level the draft model's attention for the newest rows (the shape of a 68M Llama draft: 2 layers, 12 heads of
    64) and the stop decision, whose flag the host reads; at the decided draft length the target's 32 attention layers,
    verification and update.  One HIP graph per level and one per draft length.  The iteration as the device decides
    it is checked against the same sequence composed from the oracle; the time per iteration is reported for every
    draft length (levels forced, flags still read)."""
    import numpy as np
    import oracle
    import gpu_helpers as H
    from workloads import WORKLOADS, scaled
    w = WORKLOADS["fork"]
    wd = scaled(w, H=12, d=64, cfg_id=w.cfg_id + 200)
    seed, out_bias = 1, 0.8                   # the stand-in decision model's outputs straddle beta at level 2 with this bias
    it = H.DynamicIteration(binding, w, wd, 2, N_LAYERS, seed, out_bias)
    levels, targets = it.capture()
    gamma, flags = it.run(lambda g: levels[g].replay(), lambda g: targets[g].replay())
    got = it.snapshot(gamma)
    # ---- the oracle's side of the same iteration ----
    vi, off, V = it.vi, it.off, w.V
    want_gamma = it.D
    for g in range(1, it.D):
        rows = vi["q_draft"][:, 1 + off[g - 1]:1 + off[g]]
        pr = oracle.mlp(it.ws_host, it.bs_host, oracle.decision_features(rows.reshape(-1, V), it.K)).reshape(w.B, it.W)
        st = oracle.early_stop(pr, it.BETA)
        assert np.abs(pr - it.BETA).min() > 1e-5 and np.array_equal(flags[g - 1], st), f"stop decision of level {g} differs from the oracle"
        if st.all():
            want_gamma = g
            break
    assert gamma == want_gamma, "the device stopped drafting at another level than the oracle"
    n = off[gamma]
    M = oracle.build_mask(w.branching)
    H.assert_close(got["draft_out"][0].astype(np.float64), oracle.tree_attention(it.draft_host[0], M, n), "bf16", "dynamic: draft layer 0")
    H.assert_close(got["target_out"][0].astype(np.float64), oracle.tree_attention(it.target_host[0], M, n), "bf16", "dynamic: target layer 0")
    tokens = np.ascontiguousarray(vi["tokens"][:, :n])
    want = oracle.verify_tree(0, w.branching[:gamma], tokens, np.ascontiguousarray(vi["p_target"][:, :1 + n]),
                              np.ascontiguousarray(vi["q_draft"][:, :1 + off[gamma - 1]]),
                              np.ascontiguousarray(vi["u_accept"][:, :n]), vi["u_sample"])
    assert all(np.array_equal(got[k], x) for k, x in zip(("path", "alen", "new"), want)), "dynamic: verification differs from the oracle"
    kp, vp, new_lens = oracle.commit_path(it.target_host[0], gamma, n, want[0], want[1])
    assert np.array_equal(got["caches"][0][0].view(kp.dtype), kp) and np.array_equal(got["caches"][0][1].view(vp.dtype), vp) \
        and np.array_equal(got["lens"], new_lens), "dynamic: caches after the update differ from the oracle"
    want_ids, want_n = oracle.commit_ids(gamma, tokens, want[0], want[1], want[2], 1)
    assert np.array_equal(got["ids"], want_ids) and np.array_equal(got["n_ids"], want_n)
    # ---- time per iteration by draft length ----
    by_gamma = {}
    lf, tf = (lambda g: levels[g].replay()), (lambda g: targets[g].replay())
    for g in range(1, it.D + 1):
        for _ in range(5):
            it.run(lf, tf, force_gamma=g, caches=False)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(iterations):
            it.run(lf, tf, force_gamma=g, caches=False)
        torch.cuda.synchronize()
        t_all = (time.perf_counter() - t0) / iterations
        t0 = time.perf_counter()
        for _ in range(iterations):
            targets[g].replay()
        torch.cuda.synchronize()
        t_target = (time.perf_counter() - t0) / iterations
        by_gamma[f"gamma{g}"] = {"tree_tokens": off[g], "ms_per_iteration": round(t_all * 1e3, 4),
                                 "of_which_target_step_ms": round(t_target * 1e3, 4),
                                 "draft_levels_and_decisions_ms": round((t_all - t_target) * 1e3, 4),
                                 "tree_tokens_per_s": round(w.B * off[g] / t_all, 1)}
    return {"workload": f"fork: B{w.B} H{w.H} d{w.d} bf16 prefix {w.prefix_max} tree {w.branching} V={V}; draft attention "
                        f"2 layers x {wd.H} heads of {wd.d}; decision model top-{it.K} + entropy -> 64 -> 1, beta {it.BETA}",
            "decided_on_device": {"gamma": int(gamma), "stop_flags_by_level": [int(f[0]) for f in flags],
                                  "accept_len": int(got["alen"][0]), "verified_vs_oracle":
                                  "stop flags, one draft and one target layer in full, verification, updated cache, ids"},
            "launch": "one HIP graph per level (draft attention + decision), one per draft length (32 target layers + "
                      "verification + update); the host reads the 4-byte stop flag after each level",
            "iterations_timed": iterations, "by_draft_length": by_gamma}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=100)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--workload", default="cfg2")
    ap.add_argument("--extra", default="cfg1,cfg3,cfg4,cfg5,cfg4_b64",
                    help="other configurations reported beside the headline one (attention roofline, verification, "
                         "oracle baseline; cfg1 and cfg3 also as whole steps; cfg5 at gamma 5 and 4)")
    ap.add_argument("--kernel-reps", type=int, default=64)
    ap.add_argument("--extra-reps", type=int, default=200,
                    help="timed launches (after as many untimed ones) of each large configuration's attention")
    ap.add_argument("--gqa-kv-heads", type=int, default=8,
                    help="key/value heads of the grouped-query variant of cfg4 (0 skips that section)")
    ap.add_argument("--verify-batch", type=int, default=128,
                    help="sequences of the batched verification section (0 skips it)")
    ap.add_argument("--decision-batch", type=int, default=64,
                    help="trees per call in the early-stop decision-model section (0 = skip)")
    ap.add_argument("--dynamic-iterations", type=int, default=50,
                    help="timed iterations per draft length of the dynamic-setting section on the fork-shaped tree (0 skips it)")
    ap.add_argument("--no-fp8kv", action="store_true", help="skip the fp8 prefix-cache variants of cfg4 / cfg5")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--eager", action="store_true", help="launch the step's kernels one by one instead of replaying a HIP graph")
    ap.add_argument("--replay-only", type=int, default=0,
                    help="for profilers: capture the headline step, replay it this many times and exit")
    ap.add_argument("--key-splits", type=int, default=0,
                    help="measurement sweeps: key splits of the headline workload's attention (0 = the library's plan)")
    ap.add_argument("--stages", type=int, default=0, help="measurement sweeps: LDS stages of the bf16 K/V ring (0 = the library's plan)")
    ap.add_argument("--tree-keys", type=int, default=0,
                    help="measurement sweeps: which workgroup takes the tree's own keys (0 = the library's plan, 1 own, 2 first split, 3 last split)")
    ap.add_argument("--fold-kernel", action="store_true",
                    help="measurement sweeps: fold the key splits' partial results in a second kernel")
    ap.add_argument("--traffic-calibration", action="store_true",
                    help="only run a 1 GiB device-to-device copy a few times (the known-size kernel that the "
                         "FETCH_SIZE / WRITE_SIZE counters of a rocprofv3 --pmc run are scaled by) and exit")
    args = ap.parse_args()
    if args.gpus != 1:
        sys.exit("bench.py: this build measures one GPU only (the path shards by sequence and head without any "
                 "exchange, so N GPUs are N independent copies of this run); run with --gpus 1")
    import torch
    assert torch.cuda.is_available(), "bench.py needs the MI355X"
    torch.cuda.set_device(0)
    if args.traffic_calibration:
        src = torch.ones(1 << 28, dtype=torch.float32, device="cuda")      # 1 GiB read + 1 GiB written per copy
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"calibration": "3 device-to-device copies", "bytes_read_each": src.numel() * 4,
                          "bytes_written_each": src.numel() * 4}))
        return
    import numpy as np
    from paper_2409_10644_amd import binding
    import gpu_helpers as H
    import oracle
    from workloads import WORKLOADS
    hip = binding.HipRuntime()
    traffic = measured_traffic()

    w_name = args.workload
    w = WORKLOADS[w_name]
    kv_bytes = w.B * w.H * w.prefix_max * w.d * (2 if w.dtype == "bf16" else 4) * 2
    n_sets = N_LAYERS if kv_bytes * N_LAYERS <= (8 << 30) else max(1, min(N_LAYERS, (2 << 30) // kv_bytes))
    tuning = None
    if args.key_splits or args.fold_kernel or args.stages or args.tree_keys:
        tuning = binding.AttentionTuning(key_splits=args.key_splits, fold=1 if args.fold_kernel else 0, stages=args.stages,
                                         tree_keys=args.tree_keys)
    # the verification draw of the timed step: a typical one (see pick_verify_seed), not whatever seed 0 gives
    v_seed, seed_inputs, seed_lens = pick_verify_seed(w, w.gamma_max, w.mode)
    st = Step(w_name, n_sets, tuning=tuning, verify_seed=v_seed)
    alpha, t_attn_cpu = st.check_against_oracle()
    log(f"[bench] {w_name}: outputs verified against the oracle; verification seed {v_seed} (accepted length "
        f"{alpha:.2f}, mean over seeds {np.mean(seed_lens):.2f})")
    if args.replay_only:
        ms, launch, n_ramp, graph = timed_steps(st, torch, args.replay_only, args.warmup, False)
        print(json.dumps({"replayed": args.replay_only, "ms_per_step": round(ms, 4), "launch": launch}))
        return

    ms_per_step, launch, n_ramp, graph = timed_steps(st, torch, args.steps, args.warmup, args.eager)
    value = w.B * st.n / (ms_per_step * 1e-3)

    roof = roofline_of(st, hip, args.kernel_reps, traffic, warm=args.kernel_reps)
    # the same launch on ONE K/V set over and over: the 16 MiB of a small workload then come from the 256 MB
    # last-level cache, not from HBM.  Reported beside the cold figure (which rotates over n_sets sets), never as it.
    warm_avg = time_kernel(st, hip, binding.KERNEL_ATTN_SWEEP, lambda i: st.attention(0), args.kernel_reps, warm=10)[0]
    roof["warm_cache_launch_us"] = round(warm_avg * 1e3, 2)
    has_fold_kernel = st.plan.key_splits > 1 and not st.plan.fold_in_kernel
    m_avg = time_kernel(st, hip, binding.KERNEL_ATTN_MERGE, lambda i: st.attention(i), args.kernel_reps)[0] if has_fold_kernel else 0.0
    vsec = verify_section(st, hip, args.kernel_reps)
    # the walk over all the seeds the timed one was picked from: mean time per call and per visited context
    per_seed = []
    for s, vi in enumerate(seed_inputs):
        st.set_verify_inputs(s, vi)
        def cold_verify(i):
            flush_caches(torch, i)
            st.verify()
        t = time_kernel(st, hip, binding.KERNEL_VERIFY_WALK, cold_verify, 8, warm=1)[0]
        torch.cuda.synchronize()
        al = st.alen.cpu().numpy()
        per_seed.append((t * 1e3, int(np.minimum(al + 1, st.gamma).sum()), float(al.mean())))
    st.set_verify_inputs(v_seed, seed_inputs[v_seed])
    vsec["over_seeds"] = {"seeds": len(per_seed), "mean_launch_us": round(float(np.mean([x[0] for x in per_seed])), 2),
                          "min_launch_us": round(min(x[0] for x in per_seed), 2), "max_launch_us": round(max(x[0] for x in per_seed), 2),
                          "mean_us_per_visited_context": round(float(np.sum([x[0] for x in per_seed]) / np.sum([x[1] for x in per_seed])), 2),
                          "mean_accept_len": round(float(np.mean([x[2] for x in per_seed])), 3),
                          "alpha": round(float(np.mean([x[2] for x in per_seed])) / st.gamma, 3),
                          "accept_len_by_seed": [round(x[2], 2) for x in per_seed]}
    out = {
        "metric": "verified tree-tokens/s, whole verification step (32 tree-attention layers + acceptance)",
        "value": round(value, 1), "unit": "tree-tokens/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": w.dtype, "data": "synthetic",
        "config": {"workload": f"{w_name}: B{w.B} H{w.H} d{w.d} {w.dtype} prefix {w.prefix_min}"
                               f"{'' if w.prefix_min == w.prefix_max else '-' + str(w.prefix_max)} tree {w.branching} "
                               f"N={st.n} gamma={st.gamma} V={w.V} mode={'target' if st.mode else 'draft'}-init",
                   "layers_per_step": N_LAYERS, "kv_sets": n_sets, "launch": launch,
                   "untimed_steps_before": n_ramp, "verified_vs_oracle": True, "verify_seed": v_seed,
                   "mean_accept_len": round(alpha, 3)},
        "roofline": roof,
        # verify_walk: caches overwritten before the launch; verify_walk_in_step: what the walk adds to the replayed
        # step, i.e. the step minus its 32 sweeps timed the same way (replays of a graph, launch gap included in both)
        "kernels_us": {"attn_sweep": roof["avg_launch_us"], "attn_merge": round(m_avg * 1e3, 2),
                       "verify_walk": vsec["avg_launch_us"],
                       "verify_walk_in_step": round(ms_per_step * 1e3 - N_LAYERS * roof["avg_launch_us"], 2)
                       if launch == "hip-graph" and roof.get("timed", "").startswith("one HIP event pair around") else None},
        "verify_roofline": vsec,
    }
    # the same verification for candidates drawn without replacement (a scheme next to the paper's), same shapes
    try:
        from workloads import verify_inputs
        vi2 = verify_inputs(w, seed=v_seed, gamma=st.gamma, mode=st.mode, replacement=False)
        d2 = [H.dev(vi2[k]) for k in ("tokens", "p_target", "q_draft", "u_accept", "u_sample")]
        o2 = [torch.zeros_like(st.path), torch.zeros_like(st.alen), torch.zeros_like(st.new)]

        def v2call(i):
            binding.verify_tree_sampling(st.view, st.mode, binding.MCSD_WITHOUT_REPLACEMENT, w.B, w.V, d2[0], d2[1], d2[2],
                                         vi2["p_target"].shape[1] * w.V, vi2["q_draft"].shape[1] * w.V, d2[3], d2[4],
                                         st.n_new, o2[0], o2[1], o2[2], st.vws)
        v2call(0)
        torch.cuda.synchronize()
        want2 = oracle.verify_tree(st.mode, w.branching[:st.gamma], vi2["tokens"], vi2["p_target"], vi2["q_draft"],
                                   vi2["u_accept"], vi2["u_sample"], replacement=False)
        got2 = (o2[0].cpu().numpy(), o2[1].cpu().numpy(), o2[2].cpu().numpy()[:, :st.n_new])
        assert all(np.array_equal(a, b) for a, b in zip(got2, want2)), "without-replacement verification differs from the oracle"
        def v2cold(i):
            flush_caches(torch, i)
            v2call(i)
        v2_avg = time_kernel(st, hip, binding.KERNEL_VERIFY_WALK, v2cold, 24, warm=2)[0]
        out["kernels_us"]["verify_walk_without_replacement"] = round(v2_avg * 1e3, 2)
        out["verify_without_replacement"] = {"avg_launch_us": round(v2_avg * 1e3, 2), "verified_vs_oracle": True,
                                             "mean_accept_len": round(float(want2[1].mean()), 3)}
    except Exception as ex:
        out["verify_without_replacement"] = {"error": repr(ex)}
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(st, t_attn_cpu)
    # the draft side of the loop: attention for the newest level only, a fresh slice of the mask per level
    lvl = {}
    lvl_ws = binding.new_workspace(max(binding.tree_attention_rows_workspace(w.B, w.H, w.d, binding.slice_mask(st.mask, g).n_nodes,
                                                                           int(binding.slice_mask(st.mask, g).level_off_host[g - 1]), st.cap)
                                       for g in range(1, st.gamma + 1)))
    for g in range(1, st.gamma + 1):
        vg = binding.slice_mask(st.mask, g)
        rb = int(vg.level_off_host[g - 1])

        def level_call(i, vg=vg, rb=rb):
            a = st.layers[i % len(st.layers)]
            binding.tree_attention_rows(vg, a.code, w.B, w.H, w.d, rb, a.q, a.kt, a.vt, a.node_stride, a.kp, a.vp, a.base,
                                        a.lens, a.head_stride, st.cap, a.scale, a.out, lvl_ws)
        for i in range(8):
            level_call(i)
        torch.cuda.synchronize()
        t0l = time.perf_counter()
        for i in range(64):
            level_call(i)
        torch.cuda.synchronize()
        lvl[f"gamma{g}_rows{vg.n_nodes - rb}"] = round((time.perf_counter() - t0l) / 64 * 1e6, 1)
    out["level_attention_call_us"] = lvl
    # The row after the step: the accepted path appended to every layer's cache (last: it overwrites cache rows).
    # Timed with the walk's own result and with a full path forced into the outputs (every level accepted: gamma rows
    # of every head of every layer move), so that the copy kernel is never timed on an empty path only.
    ids = torch.zeros((w.B, st.gamma + 1), dtype=torch.int32, device="cuda")
    n_ids = torch.zeros((w.B,), dtype=torch.int32, device="cuda")
    lens_c = st.layers[0].lens.clone()
    st.verify()
    torch.cuda.synchronize()
    commit = {"layers_per_call": len(st.layers)}
    own = (st.path.clone(), st.alen.clone())
    sizes = oracle.level_sizes(w.branching[:st.gamma])
    chain = torch.tensor(sizes.cumsum() - sizes, dtype=torch.int32, device="cuda")   # first node of every level: a root-to-leaf path
    for tag, (pth, aln) in (("walk_result", own), ("full_path", (chain.repeat(w.B, 1), torch.full_like(st.alen, st.gamma)))):
        st.path.copy_(pth)
        st.alen.copy_(aln)

        def commit_once(i):
            lens_c.copy_(st.layers[0].lens)
            st.commit(lens_c, ids, n_ids)
        c_avg = time_kernel(st, hip, binding.KERNEL_COMMIT_COPY, commit_once, 20, warm=5)[0]
        torch.cuda.synchronize()
        t0c = time.perf_counter()
        for i in range(20):
            commit_once(i)
        torch.cuda.synchronize()
        call_us = (time.perf_counter() - t0c) / 20 * 1e6
        rows = float(aln.float().mean().item())
        commit[tag] = {"accept_len": round(rows, 3), "copy_kernel_us": round(c_avg * 1e3, 2),
                       "call_us_with_length_reset": round(call_us, 1),
                       "bytes_moved": int(rows * w.B * len(st.layers) * w.H * w.d * 2 * 2 * 2)}
    out["commit_path"] = commit
    del st, graph
    torch.cuda.empty_cache()

    extra = {}
    plans = {"cfg1": dict(n_sets=N_LAYERS, with_step=True), "cfg3": dict(n_sets=16, with_step=True),
             "cfg5": dict(gammas=(5, 4))}
    for name in [x for x in args.extra.split(",") if x and x != w_name]:
        try:
            extra.update(config_section(name, hip, args, traffic, **plans.get(name, {})))
        except Exception as ex:      # an extra workload must not lose the headline line
            extra[name] = {"error": repr(ex)}
    # grouped-query variant of the ragged batch (beyond the paper's multi-head shape): 32 query heads on 8 kv heads
    if args.gqa_kv_heads > 0 and "cfg4" in args.extra:
        try:
            from workloads import scaled, attention_inputs, prefix_lens
            wq = WORKLOADS["cfg4"]
            Hkv = args.gqa_kv_heads
            wk = scaled(wq, H=Hkv, cfg_id=wq.cfg_id + 100)
            lens = prefix_lens(wq, 0)
            qi = attention_inputs(wq, seed=0, lens=lens, kv_capacity=int(wq.prefix_max))
            ki = attention_inputs(wk, seed=0, lens=lens, kv_capacity=int(wq.prefix_max))
            aq, ak = H.AttnDevice(qi), H.AttnDevice(ki)
            vg = binding.slice_mask(binding.build_mask(wq.branching), wq.gamma_max)
            n = vg.n_nodes
            wsb = binding.tree_attention_gqa_workspace(wq.B, wq.H, Hkv, wq.d, n, 0, int(wq.prefix_max))
            wsg = binding.new_workspace(wsb)

            def gcall(i):
                binding.tree_attention_gqa(vg, 1, wq.B, wq.H, Hkv, wq.d, 0, aq.q, ak.kt, ak.vt, ak.node_stride, ak.kp, ak.vp,
                                           ak.base, ak.lens, ak.head_stride, int(wq.prefix_max), aq.scale, aq.out, wsg)
            aq.out.fill_(float("nan"))
            gcall(0)
            torch.cuda.synchronize()
            G = wq.H // Hkv
            cap = ki["k_prefix"].shape[2]
            rep_ = dict(qi, k_tree=np.repeat(ki["k_tree"], G, axis=1), v_tree=np.repeat(ki["v_tree"], G, axis=1),
                        k_prefix=np.repeat(ki["k_prefix"], G, axis=1), v_prefix=np.repeat(ki["v_prefix"], G, axis=1),
                        head_stride=cap * wq.d, seq_base=(np.arange(wq.B, dtype=np.int64) * (wq.H * cap * wq.d)))
            got = aq.out[:, :, :n].float().cpu().numpy().astype(np.float64)
            H.assert_close(got, oracle.tree_attention(rep_, oracle.build_mask(wq.branching), n), "bf16", "bench gqa, every element")
            del rep_

            gs = Ctx(binding, torch)
            g_avg, g_med, g_p10, g_p90 = time_kernel(gs, hip, binding.KERNEL_ATTN_SWEEP, gcall, args.extra_reps, warm=args.extra_reps)
            torch.cuda.synchronize()
            time.sleep(0.05)
            g_idle = time_kernel(gs, hip, binding.KERNEL_ATTN_SWEEP, gcall, 3)[0]
            gbytes = sum(2 * wq.d * (Hkv * (2 * int(L) + 2 * n) + wq.H * 2 * n) for L in lens)
            gflops = sum(wq.H * 4 * n * (int(L) + n) * wq.d for L in lens)
            gp = binding.tree_attention_plan(None, 1, 0, wq.B, wq.H, Hkv, wq.d, n, 0, int(wq.prefix_max))
            extra["cfg4_gqa"] = {"bound": "mfma", "kernel": f"tree_attn_bf16_kernel<{wq.d}, {gp.query_blocks}, {gp.stages}, false>",
                                 "workgroups": int(gp.workgroups), "fold_in_kernel": bool(gp.fold_in_kernel),
                                 "achieved": round(gflops / (g_avg * 1e-3) / 1e12, 1),
                                 "peak": MFMA_BF16_PEAK_TFLOPS, "unit": "TFLOP/s", "frac": round(gflops / (g_avg * 1e-3) / 1e12 / MFMA_BF16_PEAK_TFLOPS, 4),
                                 "traffic": None, "flops_per_launch": int(gflops), "algorithmic_bytes_per_launch": int(gbytes),
                                 "hbm_GBps": round(gbytes / (g_avg * 1e-3) / 1e9, 1), "avg_launch_us": round(g_avg * 1e3, 2),
                                 "p10_us": round(g_p10 * 1e3, 2), "p90_us": round(g_p90 * 1e3, 2), "launches_timed": args.extra_reps,
                                 "launch_after_idle_us": round(g_idle * 1e3, 2),
                                 "verified_vs_oracle": "every element",
                                 "workload": f"cfg4 with {wq.H} query heads on {Hkv} key/value heads (B{wq.B} N={n})"}
            del aq, ak
            torch.cuda.empty_cache()
        except Exception as ex:
            extra["cfg4_gqa"] = {"error": repr(ex)}
    # the same sweeps over an fp8 (E4M3) prefix cache (beyond the paper's bf16 setting): half the prefix bytes
    if not args.no_fp8kv:
        for name in [x for x in args.extra.split(",") if x in ("cfg4", "cfg5")]:
            try:
                from workloads import attention_inputs, prefix_lens
                w8 = WORKLOADS[name]
                lens = prefix_lens(w8, 0)
                cap = int(w8.prefix_max)
                inp8 = attention_inputs(w8, seed=0, kv_capacity=cap, kv_fp8=(0.5, 0.25))
                q8, kt8, vt8 = (H.dev(inp8[k], "bf16") for k in ("q", "k_tree", "v_tree"))
                kp8, vp8 = torch.from_numpy(inp8["k_prefix"]).cuda(), torch.from_numpy(inp8["v_prefix"]).cuda()
                lens8 = H.dev(np.ascontiguousarray(inp8["lens"], dtype=np.int32))
                base8 = H.dev(np.ascontiguousarray(inp8["seq_base"], dtype=np.int64))
                out8 = torch.full(q8.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
                v8 = binding.slice_mask(binding.build_mask(w8.branching), w8.gamma_max)
                n8 = v8.n_nodes
                ws8 = binding.new_workspace(binding.tree_attention_fp8kv_workspace(w8.B, w8.H, w8.H, n8, 0, cap))

                def fcall(i):
                    binding.tree_attention_fp8kv(v8, w8.B, w8.H, w8.H, 0, q8, kt8, vt8, inp8["node_stride"],
                                                 kp8, vp8, inp8["k_scale"], inp8["v_scale"], base8, lens8, inp8["head_stride"],
                                                 cap, float(np.float32(inp8["scale"])), out8, ws8)
                fcall(0)
                torch.cuda.synchronize()
                got8 = out8[:, :, :n8].float().cpu().numpy().astype(np.float64)
                H.assert_close(got8, oracle.tree_attention_fp8kv(inp8, oracle.build_mask(w8.branching), n8), "bf16",
                               "bench fp8kv, every element")

                fs = Ctx(binding, torch)
                f_avg, f_med, f_p10, f_p90 = time_kernel(fs, hip, binding.KERNEL_ATTN_SWEEP, fcall, args.extra_reps, warm=args.extra_reps)
                torch.cuda.synchronize()
                time.sleep(0.05)
                f_idle = time_kernel(fs, hip, binding.KERNEL_ATTN_SWEEP, fcall, 3)[0]
                fbytes, fflops = attention_algorithmic(w8, lens, n8, kv_bytes_per_elem=1)
                fp = binding.tree_attention_plan(None, 1, 1, w8.B, w8.H, w8.H, w8.d, n8, 0, cap)
                kname = f"tree_attn_bf16_kernel<{w8.d}, {fp.query_blocks}, {fp.stages}, true>"
                # which roof: the bytes at 8 TB/s against the flops at the dense bf16 peak
                t_hbm, t_mfma = fbytes / (HBM_PEAK_GBPS * 1e9), fflops / (MFMA_BF16_PEAK_TFLOPS * 1e12)
                issue_bound = fp.query_blocks == 4   # four query blocks: the soft-max + MFMA instruction stream, not HBM, is the limit
                entry = {"kernel": kname, "workgroups": int(fp.workgroups), "fold_in_kernel": bool(fp.fold_in_kernel),
                         "traffic": traffic.get((kname.replace(" ", ""), int(fp.workgroups))),
                         "algorithmic_bytes_per_launch": int(fbytes), "flops_per_launch": int(fflops),
                         "avg_launch_us": round(f_avg * 1e3, 2), "p10_us": round(f_p10 * 1e3, 2), "p90_us": round(f_p90 * 1e3, 2),
                         "hbm_GBps": round(fbytes / (f_avg * 1e-3) / 1e9, 1), "hbm_frac": round(fbytes / (f_avg * 1e-3) / 1e9 / HBM_PEAK_GBPS, 4),
                         "mfma_tflops": round(fflops / (f_avg * 1e-3) / 1e12, 1),
                         "mfma_frac": round(fflops / (f_avg * 1e-3) / 1e12 / MFMA_BF16_PEAK_TFLOPS, 4),
                         "time_at_hbm_peak_us": round(t_hbm * 1e6, 1), "time_at_mfma_peak_us": round(t_mfma * 1e6, 1),
                         "launches_timed": args.extra_reps, "launch_after_idle_us": round(f_idle * 1e3, 2),
                         "attn_tree_tokens_per_s": round(w8.B * n8 / (f_avg * 1e-3), 1), "verified_vs_oracle": "every element",
                         "workload": f"{name} with the prefix cache in fp8 E4M3 (B{w8.B} N={n8})"}
                if issue_bound:
                    entry.update({"bound": "mfma", "achieved": entry["mfma_tflops"], "peak": MFMA_BF16_PEAK_TFLOPS,
                                  "unit": "TFLOP/s", "frac": entry["mfma_frac"]})
                else:
                    entry.update({"bound": "hbm", "achieved": entry["hbm_GBps"], "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                                  "frac": entry["hbm_frac"]})
                extra[name + "_fp8kv"] = entry
                del kp8, vp8
                torch.cuda.empty_cache()
            except Exception as ex:
                extra[name + "_fp8kv"] = {"error": repr(ex)}
    # the vocabulary pass at a batch that fills half the chip's compute units (one workgroup per sequence)
    if args.verify_batch > 0:
        try:
            from workloads import scaled, verify_inputs
            wb = scaled(WORKLOADS[w_name], B=args.verify_batch)
            vi = verify_inputs(wb, seed=1, mode=0)
            vv = binding.slice_mask(binding.build_mask(wb.branching), wb.gamma_max)
            got = H.run_verify(binding, vv, 0, vi)
            want = oracle.verify_tree(0, wb.branching, vi["tokens"], vi["p_target"], vi["q_draft"], vi["u_accept"], vi["u_sample"])
            assert all((a == b).all() for a, b in zip(got, want)), "batched verification differs from the oracle"
            dp, dq = H.dev(vi["p_target"]), H.dev(vi["q_draft"])
            dt_, dua, dus = H.dev(vi["tokens"]), H.dev(vi["u_accept"]), H.dev(vi["u_sample"])
            o_path = torch.zeros((wb.B, vv.gamma), dtype=torch.int32, device="cuda")
            o_len = torch.zeros((wb.B,), dtype=torch.int32, device="cuda")
            o_new = torch.zeros((wb.B, 1), dtype=torch.int32, device="cuda")
            vs = Ctx(binding, torch)

            def vcall(i):
                binding.verify_tree(vv, 0, wb.B, wb.V, dt_, dp, dq, vi["p_target"].shape[1] * wb.V, vi["q_draft"].shape[1] * wb.V,
                                    dua, dus, 1, o_path, o_len, o_new, None)
            vb_warm = time_kernel(vs, hip, binding.KERNEL_VERIFY_WALK, vcall, 30, warm=10)[0]

            def vcall_cold(i):       # the 39 MB of rows this call reads would otherwise come from the last-level cache
                flush_caches(torch, i)
                vcall(i)
            vb_avg = time_kernel(vs, hip, binding.KERNEL_VERIFY_WALK, vcall_cold, 24, warm=2)[0]
            vbytes = walk_bytes(wb, vv.gamma, 0, 1, got[0], got[1])
            extra["verify_batch%d" % wb.B] = {
                "bound": "hbm", "kernel": walk_kernel(wb.V, wb.B), "achieved": round(vbytes / (vb_avg * 1e-3) / 1e9, 1),
                "peak": HBM_PEAK_GBPS, "unit": "GB/s", "frac": round(vbytes / (vb_avg * 1e-3) / 1e9 / HBM_PEAK_GBPS, 4),
                "algorithmic_bytes_per_launch": int(vbytes), "avg_launch_us": round(vb_avg * 1e3, 2),
                "rows_still_cached_launch_us": round(vb_warm * 1e3, 2),
                "sequences_per_s": round(wb.B / (vb_avg * 1e-3), 1), "mean_accept_len": round(float(got[1].mean()), 3),
                "alpha": round(float(got[1].mean()) / vv.gamma, 3),
                "verified_vs_oracle": True, "workload": f"{w_name} verification, B={wb.B}, V={wb.V}, draft-init"}
            del dp, dq
        except Exception as ex:
            extra["verify_batch"] = {"error": repr(ex)}
    # early-stop decision models (Sec. 3.3) on the newest contexts of fork-shaped trees of width 16: one tree, and a
    # batch whose rows (4 distinct copies, > 512 MB) cannot stay in the last-level cache between launches
    if args.decision_batch > 0:
        try:
            from workloads import hidden_states, mlp_weights, scaled, verify_inputs
            k, Wd, beta = 10, 16, 0.4
            Bd = args.decision_batch
            wd = scaled(WORKLOADS["fork"], B=Bd, branching=(Wd, 1))
            q = verify_inputs(wd, seed=1, mode=0)["q_draft"]                  # [Bd][1 + 16][V]; rows 1.. are the new contexts
            V = wd.V
            ws, bs = mlp_weights((k + 1, 64, 1), seed=0, out_bias=-0.3)
            mlp2 = binding.make_mlp([torch.from_numpy(a).cuda() for a in ws], [torch.from_numpy(a).cuda() for a in bs])
            wbytes = sum(a.nbytes for a in ws + bs)
            copies = 4
            rows = torch.from_numpy(np.ascontiguousarray(q[:, 1:])).cuda().repeat(copies, 1, 1)   # [copies*Bd][16][V]
            prob = torch.zeros((copies * Bd, Wd), dtype=torch.float32, device="cuda")
            stop = torch.zeros((copies * Bd,), dtype=torch.int32, device="cuda")

            ds = Ctx(binding, torch)
            nb = min(Bd, 4)
            want = oracle.mlp(ws, bs, oracle.decision_features(q[:nb, 1:].reshape(nb * Wd, V), k)).reshape(nb, Wd)
            for trees, tag in ((1, "1"), (copies * Bd, str(copies * Bd))):
                def dcall(i, trees=trees):
                    binding.early_stop_distribution(mlp2, trees, Wd, V, k, rows, Wd * V, V, beta, None, prob, stop)
                dcall(0)
                torch.cuda.synchronize()
                nchk = min(nb, trees)
                gotp = prob[:nchk].cpu().numpy()
                assert np.abs(gotp - want[:nchk]).max() <= 1e-5, "decision model differs from the oracle"
                assert stop[:nchk].cpu().tolist() == [int((gotp[b] < np.float32(beta)).all()) for b in range(nchk)]
                d_avg = time_kernel(ds, hip, binding.KERNEL_DECISION, dcall, 30, warm=10)[0]
                t0 = time.perf_counter()
                for i in range(50):
                    dcall(i)
                torch.cuda.synchronize()
                call_us = (time.perf_counter() - t0) / 50 * 1e6
                dbytes = trees * Wd * V * 4 + wbytes
                extra["early_stop_distribution_trees" + tag] = {
                    "bound": "hbm", "kernel": "decision_distribution_kernel", "achieved": round(dbytes / (d_avg * 1e-3) / 1e9, 1),
                    "peak": HBM_PEAK_GBPS, "unit": "GB/s", "frac": round(dbytes / (d_avg * 1e-3) / 1e9 / HBM_PEAK_GBPS, 4),
                    "algorithmic_bytes_per_launch": int(dbytes), "avg_launch_us": round(d_avg * 1e3, 2),
                    "call_us": round(call_us, 1), "verified_vs_oracle": True,
                    "workload": f"{trees} fork tree(s) of width {Wd}, V={V}, top-{k} + entropy, MLP {k + 1}-64-1, beta {beta}"}
            del rows
            hw = (768, 256, 64, 1)                                          # hidden width of the 68M draft model
            ws1, bs1 = mlp_weights(hw, seed=1, out_bias=-0.4)
            mlp1 = binding.make_mlp([torch.from_numpy(a).cuda() for a in ws1], [torch.from_numpy(a).cuda() for a in bs1])
            hx = hidden_states(Bd, Wd, hw[0], seed=1)
            hxd = torch.from_numpy(hx).cuda()

            def hcall(i):
                binding.early_stop_hidden(mlp1, Bd, Wd, hxd, Wd * hw[0], hw[0], beta, prob, stop)
            hcall(0)
            torch.cuda.synchronize()
            want1 = oracle.mlp(ws1, bs1, hx[:nb].reshape(nb * Wd, hw[0]).astype(np.float64)).reshape(nb, Wd)
            assert np.abs(prob[:nb].cpu().numpy() - want1).max() <= 1e-6, "hidden-state decision model differs from the oracle"
            h_avg = time_kernel(ds, hip, binding.KERNEL_DECISION, hcall, 30, warm=10)[0]
            extra["early_stop_hidden_trees%d" % Bd] = {
                "kernel": "decision_hidden_kernel", "avg_launch_us": round(h_avg * 1e3, 2), "verified_vs_oracle": True,
                "bytes_per_launch": int(hx.nbytes + sum(a.nbytes for a in ws1 + bs1)),
                "workload": f"{Bd} trees of width {Wd}, hidden width {hw[0]}, MLP {'-'.join(map(str, hw))} (latency-bound)"}
        except Exception as ex:
            extra["early_stop"] = {"error": repr(ex)}
    if args.dynamic_iterations > 0:
        try:
            out["dynamic_iteration"] = dynamic_section(binding, torch, args.dynamic_iterations)
        except Exception as ex:
            out["dynamic_iteration"] = {"error": repr(ex)}
        torch.cuda.empty_cache()
    # yardstick: what the HBM of this machine delivers to a plain read-only streaming kernel (4 GiB buffer)
    try:
        buf = torch.empty(4 << 30, dtype=torch.uint8, device="cuda")
        buf.fill_(1)
        sink = torch.zeros(16, dtype=torch.uint8, device="cuda")

        ss = Ctx(binding, torch)
        per_grid = {}
        for wgs in (192, 256, 512, 2048):      # the rate depends on how the grid's stride falls on the memory channels
            s_avg = time_kernel(ss, hip, binding.KERNEL_STREAM_READ, lambda i: binding.stream_read(buf, sink, wgs), 10, warm=10)[0]
            per_grid[wgs] = round(buf.numel() / (s_avg * 1e-3) / 1e9, 1)
        gbps = max(per_grid.values())
        out["stream_read_probe"] = {"GB/s": gbps, "frac_of_peak": round(gbps / HBM_PEAK_GBPS, 4), "bytes": buf.numel(),
                                    "GB/s_by_workgroups": per_grid}
        for r in [out["roofline"]] + [v for v in extra.values() if v.get("bound") == "hbm"]:
            r["frac_of_stream_read"] = round(r["achieved"] / gbps, 4)
        del buf
    except Exception as ex:
        out["stream_read_probe"] = {"error": repr(ex)}
    # the other yardstick: what the matrix cores of this machine sustain in a plain library GEMM (bf16, 8192^3, fp32
    # accumulation) launched back to back -- the datasheet's dense peak assumes clocks that a loaded chip does not hold
    try:
        n = 8192
        ga = torch.randn(n, n, device="cuda", dtype=torch.bfloat16)
        gb = torch.randn(n, n, device="cuda", dtype=torch.bfloat16)
        gc = torch.empty(n, n, device="cuda", dtype=torch.bfloat16)
        for _ in range(20):
            torch.matmul(ga, gb, out=gc)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(50):
            torch.matmul(ga, gb, out=gc)
        torch.cuda.synchronize()
        tf = 2.0 * n ** 3 / ((time.perf_counter() - t0) / 50) / 1e12
        out["gemm_probe"] = {"TFLOP/s": round(tf, 1), "frac_of_peak": round(tf / MFMA_BF16_PEAK_TFLOPS, 4),
                             "what": f"library bf16 GEMM {n}^3, 50 launches back to back"}
        for r in [v for v in extra.values() if v.get("bound") == "mfma"]:
            r["frac_of_gemm_probe"] = round(r["achieved"] / tf, 4)
        del ga, gb, gc
    except Exception as ex:
        out["gemm_probe"] = {"error": repr(ex)}
    # how far this machine overlaps the inner loop's matrix instructions with its vector work (no memory traffic):
    # the arrangement the sweep relies on (two wavefronts per SIMD, free-running) against the alternatives
    try:
        n_wg = torch.cuda.get_device_properties(0).multi_processor_count
        pout = torch.empty(n_wg * 512, dtype=torch.float32, device="cuda")
        iters = 2000
        names = ["one_per_simd_phases_in_turn", "two_per_simd_free_running", "two_per_simd_alternating_under_barriers",
                 "one_per_simd_software_pipelined", "two_per_simd_software_pipelined"]
        res = {}
        for sched, nm in enumerate(names):
            for _ in range(3):
                binding.issue_probe(sched, n_wg, iters, pout)
            e0, e1 = hip.event(), hip.event()
            hip.record(e0)
            for _ in range(10):
                binding.issue_probe(sched, n_wg, iters, pout)
            hip.record(e1)
            ms = hip.elapsed_ms(e0, e1) / 10
            hip.destroy(e0)
            hip.destroy(e1)
            blocks = iters * (1 if sched in (0, 3) else 2)            # 32-key blocks per SIMD and launch
            res[nm] = {"ns_per_block": round(ms * 1e6 / blocks, 1), "mfma_pipe_busy": round(blocks * 16 * 32 / 2.4e9 / (ms * 1e-3), 3)}
        out["issue_probe"] = {"what": "arithmetic of the sweep's inner loop for one 32-key block (16 MFMA 32x32x16 + soft-max of 16 "
                                      "scores per lane), no memory traffic, one workgroup per compute unit; mfma_pipe_busy assumes 32 "
                                      "cycles per MFMA at 2.4 GHz", **res}
    except Exception as ex:
        out["issue_probe"] = {"error": repr(ex)}
    # where the workgroups of a sweep-shaped grid run: dies by id, and which ids share a compute unit
    try:
        n_cu = torch.cuda.get_device_properties(0).multi_processor_count
        pl_out = torch.zeros(2 * 2 * n_cu, dtype=torch.int32, device="cuda")
        stats = []
        for _ in range(5):
            binding.placement_probe(2 * n_cu, 20000, pl_out)
            torch.cuda.synchronize()
            a = pl_out.cpu().numpy().astype(np.int64).reshape(2 * n_cu, 2)
            die, cu = a[:, 0], (a[:, 0] << 16) | (a[:, 1] & 0xff00)      # compute unit = (die, shader engine, array, cu)
            n_die = int(die.max()) + 1
            stats.append((n_die, float(np.mean(die == (die[0] + np.arange(2 * n_cu)) % n_die)), float(np.mean(cu[:n_cu] == cu[n_cu:])),
                          int(len(set(cu.tolist())))))
        out["placement_probe"] = {"workgroups": 2 * n_cu, "launches": len(stats), "dies": stats[0][0],
                                  "ids_dealt_round_robin_to_dies": round(min(s[1] for s in stats), 4),
                                  "pairs_i_and_i_plus_cus_on_one_compute_unit": round(min(s[2] for s in stats), 4),
                                  "distinct_compute_units": min(s[3] for s in stats),
                                  "what": "minimum over the launches; a grid of two sweep-shaped workgroups per compute unit"}
    except Exception as ex:
        out["placement_probe"] = {"error": repr(ex)}
    if extra:
        out["other_workloads"] = extra
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
