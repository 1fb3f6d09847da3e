#!/usr/bin/env python3
"""Depth-sparse stack throughput on one MI355X.

One step is one forward pass of the whole depth-sparse stack (router, Top-K,
gather + norm, QKV + RoPE, attention over kept tokens, output and FFN
projections, residual scatter, for every layer) over one batch of synthetic
hidden states at fixed per-layer retention. The headline workload is the
Qwen2.5-7B-shaped stack (28 x 3584, 28 q / 4 kv heads of 128, SwiGLU 18944,
batch 4 x 8192 tokens), whose retention ratios come from the allocation of
Eqs. 5-8 on similarities measured by the GPU calibration pass (the
similarity statistic of Eq. 4 on the dense stack, timed separately as
`calibration_ms`).

Inputs are resident in HBM before the timed region: every timed step runs on
its own pristine copy of the hidden states, prepared beforehand.

Prints one JSON line. `roofline` is for the kernel kind that takes the most
GPU time per step (found by an instrumented pass before the timed region),
timed with HIP events around each of its launches inside the timed region.
`cpu_baseline` times the CPU oracle on one layer of one sequence at the full
shape and extrapolates to the stack with the analytic FLOP model. The other
workloads (GPT-NeoX-160M, Qwen2.5-0.5B, the GPT-NeoX-1.4B retention sweep and
the paper's own model shapes at r = 0.9 / 0.8 / 0.7) are extra keys.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "depth-sparse stack tokens/sec at fixed r_l; MFMA util % and HBM GB/s % of peak"
PEAK_BF16_TFLOPS = 2500.0   # MI355X dense bf16 MFMA
PEAK_HBM_GBS = 8000.0       # MI355X HBM3E


# HBM traffic of the dominant kernel, from two rocprofv3 passes (FETCH_SIZE,
# then WRITE_SIZE, per dispatch) scaled by what the same counters read for the
# library's plain copy kernel of known size. A figure holds only for the
# workload, kernel kind and GEMM source it was measured on (SHA-256 of
# kernels_gemm.hip); for anything else `traffic` is null.
TRAFFIC_MEASURED = [
    # 28-layer Qwen2.5-7B-shaped stack, B 4 x T 8192, SwiGLU gate|up launch:
    # mean over the 112 sparse dispatches of 4 steps; FETCH_SIZE 3811891.2 KiB
    # x 1.9998 (copy: 114698.1 KiB read for 229376 KiB copied), WRITE_SIZE
    # 606134.0 KiB x 1.0 (equal to the bytes the launch stores). The counters
    # count L2 misses, served by the 256 MB MALL or HBM.
    {"workload": "qwen7b", "kind": "gemm_up", "bytes_per_launch": 8.4269e9,
     "gemm_source_sha256": "e891f72dd6b0f67ab29d8acfa44c4da5f7df036b942b4ea18a006e0e1214cc36",
     "profile": "profiles/gemm_up_qwen7b_traffic.md"},
]


def gemm_source_sha256():
    import hashlib
    path = os.path.join(ROOT, "paper_2607_21291_amd", "csrc", "kernels_gemm.hip")
    with open(path, "rb") as f:
        return hashlib.sha256(f.read()).hexdigest()


def measured_traffic(workload, kind):
    sha = gemm_source_sha256()
    for t in TRAFFIC_MEASURED:
        if t["workload"] == workload and t["kind"] == kind and t["gemm_source_sha256"] == sha:
            return t["bytes_per_launch"]
    return None


def log(msg):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def retention(P, w, calib_s=None):
    if w.retention is not None:
        return list(w.retention)
    s = calib_s if w.similarity is None else list(w.similarity)
    return P.retention_from_similarity(s, w.target, w.tau)


def streaming_rates(P, C, w, k, dev, weights0, reps=3):
    """The HBM-bound entry points standalone, against HBM peak: router, Top-K,
    gather, scatter and the similarity statistic, on one layer's shapes
    (B, T, d, k). "cold": each launch reads its own input buffer, cycling
    through copies that together exceed 1 GiB (more than the 256 MB MALL),
    so reads come from HBM; "hot": every launch on the same buffer."""
    import torch
    B, T, d = w.batch, w.seq, w.d_model
    eb = 4 if w.dtype == "f32" else 2
    xbytes = B * T * d * eb
    R = max(4, -(-(1 << 30) // xbytes) + 1)
    xs = [torch.randn(B, T, d, device=dev).mul_(0.02).to(w.torch_dtype) for _ in range(R)]
    scs = [torch.randn(B, T, device=dev) for _ in range(R)]
    idx = torch.stack([torch.sort(torch.randperm(T, device=dev)[:k])[0] for _ in range(B)]).to(torch.int32)
    delta = torch.randn(B, k, d, device=dev).mul_(0.02).to(w.torch_dtype)
    gout = torch.empty(B, k, d, device=dev, dtype=w.torch_dtype)
    scores = torch.empty(B, T, device=dev)
    idx_out = torch.empty(B, k, dtype=torch.int32, device=dev)
    accum = torch.zeros(2, dtype=torch.float64, device=dev)
    simws = torch.empty(max(P.sim_workspace_size(B * T), 256), dtype=torch.uint8, device=dev)
    W = {key: (v.to(dev) if hasattr(v, "to") else v) for key, v in weights0.items()
         if key.startswith("router_")}
    ops = {
        "router": (lambda i: P.router_score(xs[i], W["router_w1"], W["router_b1"], W["router_w2"],
                                            float(W["router_b2"]), scores), C.router_bytes(w, B, T)),
        "topk": (lambda i: P.topk_select(scs[i], k, idx_out), C.topk_bytes(w, B, T, k)),
        "gather": (lambda i: P.gather_rows(xs[i], idx, gout), 2.0 * eb * B * k * d + 4.0 * B * k),
        "scatter": (lambda i: P.scatter_residual(xs[i], delta, idx), 3.0 * eb * B * k * d + 4.0 * B * k),
        "sim": (lambda i: P.sim_stats(xs[i], xs[(i + 1) % R], accum, workspace=simws), C.sim_bytes(w, B, T)),
    }
    out = {}
    for name, (fn, nbytes) in ops.items():
        res = {"bytes_per_launch": nbytes}
        for mode in ("cold", "hot"):
            for i in range(min(R, 4)):
                fn(i if mode == "cold" else 0)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            n = R * reps
            torch.cuda.synchronize()
            e0.record()
            for i in range(n):
                fn(i % R if mode == "cold" else 0)
            e1.record()
            torch.cuda.synchronize()
            us = e0.elapsed_time(e1) * 1e3 / n
            gbs = nbytes / (us * 1e-6) / 1e9
            res[mode] = {"us": us, "GB/s": gbs, "frac_of_hbm_peak": gbs / PEAK_HBM_GBS}
        out[name] = res
    del xs, scs
    torch.cuda.empty_cache()
    return out


def _timed(fn, n_calls, reps_of):
    """Mean microseconds per call of fn(i) over n_calls calls (torch events)."""
    import torch
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record()
    for i in range(n_calls):
        fn(reps_of(i))
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) * 1e3 / n_calls


def router_pathway(P, C, w, ks, dev, desc, weights, x0, ws, ms_plain, steps, weights0):
    """The training-side router-score pathway (Section 3.4): the score-gated
    stack against the plain one, and the gate score gradient and the router
    backward standalone on one layer's shapes, cold (inputs cycled through
    more than 1 GiB of copies) and hot."""
    import torch
    B, T, d = w.batch, w.seq, w.d_model
    eb = 4 if w.dtype == "f32" else 2
    out = {}
    # gated stack, same k per layer
    xg = [x0.clone() for _ in range(steps)]
    xw = x0.clone()
    P.stack_forward(desc, weights, ks, xw, ws, flags=P.FLAG_GATE)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(steps):
        P.stack_forward(desc, weights, ks, xg[i], ws, flags=P.FLAG_GATE)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / steps
    out["gated_stack"] = {"ms_per_step": ms, "tokens_per_s": B * T / (ms / 1e3), "vs_plain": ms / ms_plain}
    del xg, xw
    # gate score gradient at the mean k
    k = int(round(sum(ks) / len(ks)))
    rows = B * T * d * eb
    R = max(4, -(-(1 << 30) // (3 * rows)) + 1)
    dys = [torch.randn(B, T, d, device=dev).to(w.torch_dtype) for _ in range(R)]
    xis = [torch.randn(B, T, d, device=dev).to(w.torch_dtype) for _ in range(R)]
    xos = [torch.randn(B, T, d, device=dev).to(w.torch_dtype) for _ in range(R)]
    sc = torch.randn(B, T, device=dev)
    idx = torch.stack([torch.sort(torch.randperm(T, device=dev)[:k])[0] for _ in range(B)]).to(torch.int32)
    dsc = torch.empty(B, T, device=dev)
    fn = lambda i: P.gate_score_grad(dys[i], xis[i], xos[i], sc, idx, dsc)
    nbytes = C.gate_grad_bytes(w, B, T, k)
    res = {"k": k, "bytes_per_call": nbytes}
    for mode in ("cold", "hot"):
        fn(0)
        us = _timed(fn, 3 * R, (lambda i: i % R) if mode == "cold" else (lambda i: 0))
        res[mode] = {"us": us, "GB/s": nbytes / (us * 1e-6) / 1e9, "frac_of_hbm_peak": nbytes / (us * 1e-6) / 1e9 / PEAK_HBM_GBS}
    out["gate_score_grad"] = res
    del dys, xis, xos
    # router backward over every token of the batch
    n = B * T
    W = {key: v.to(dev) for key, v in weights0.items() if key.startswith("router_") and hasattr(v, "to")}
    R = max(4, -(-(1 << 30) // (2 * rows)) + 1)
    xr = [torch.randn(B, T, d, device=dev).mul_(0.02).to(w.torch_dtype) for _ in range(R)]
    dxr = [torch.zeros(B, T, d, device=dev, dtype=w.torch_dtype) for _ in range(R)]
    dsr = torch.randn(n, device=dev)
    g = {name: torch.empty(shape, device=dev) for name, shape in
         (("dw1", (w.d_router, d)), ("db1", (w.d_router,)), ("dw2", (w.d_router,)), ("db2", (1,)))}
    rws = torch.empty(P.router_backward_workspace_size(n, d, w.d_router), dtype=torch.uint8, device=dev)
    fn = lambda i: P.router_backward(xr[i], W["router_w1"], W["router_b1"], W["router_w2"], dsr, g["dw1"], g["db1"],
                                     g["dw2"], g["db2"], dx=dxr[i], workspace=rws)
    nbytes, nflops = C.router_bwd_bytes(w, n), C.router_bwd_flops(w, n)
    res = {"n_tokens": n, "bytes_per_call": nbytes, "flops_per_call": nflops}
    for mode in ("cold", "hot"):
        fn(0)
        us = _timed(fn, 3 * R, (lambda i: i % R) if mode == "cold" else (lambda i: 0))
        res[mode] = {"us": us, "GB/s": nbytes / (us * 1e-6) / 1e9, "frac_of_hbm_peak": nbytes / (us * 1e-6) / 1e9 / PEAK_HBM_GBS,
                     "TFLOP/s": nflops / (us * 1e-6) / 1e12}
    # the three launches of one call, on the library's event timing
    P.timing_enable(64, ["backward"])
    for i in range(8):
        fn(i % R)
    torch.cuda.synchronize()
    nb, msb = P.timing_read("backward")
    P.timing_enable(0)
    res["timed_calls"] = {"calls": nb, "us_per_call": msb * 1e3 / max(nb, 1)}
    out["router_backward"] = res
    del xr, dxr
    torch.cuda.empty_cache()
    return out


# vocabulary sizes of the two model families (logit rows of Eq. 10)
VOCAB = {"neox_parallel": 50304, "qwen_seq": 151936}


def alignment_objective(P, C, w, ks, dev, desc, weights, x0, ms_plain, steps):
    """Section 3.5: the dense-teacher / sparse-student stack with Eq. 9 per
    layer, against the sparse stack alone; and the Eq. 9 and Eq. 10 kernels
    standalone (Eq. 10 on synthetic logits of the model family's vocabulary
    for every token of the batch)."""
    import torch
    B, T, d = w.batch, w.seq, w.d_model
    eb = 4 if w.dtype == "f32" else 2
    dcode = P.F32 if w.dtype == "f32" else P.BF16
    out = {}
    ws = torch.empty(P.align_stack_workspace_size(desc, dcode, B, T), dtype=torch.uint8, device=dev)
    hid = torch.zeros(w.n_layers, dtype=torch.float64, device=dev)
    xs, xt = x0.clone(), x0.clone()
    P.align_stack_forward(desc, weights, ks, xs, xt, hid, ws)
    n_steps = max(2, steps)
    pairs = [(x0.clone(), x0.clone()) for _ in range(n_steps)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for a, b in pairs:
        P.align_stack_forward(desc, weights, ks, a, b, hid, ws)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / n_steps
    out["align_stack"] = {"ms_per_step": ms, "tokens_per_s": B * T / (ms / 1e3), "vs_sparse_stack": ms / ms_plain,
                          "note": "dense teacher + sparse student + Eq. 9 per layer"}
    del pairs, ws
    # Eq. 9 kernel standalone, cold (inputs cycled through > 1 GiB) and hot
    n = B * T
    nbytes = C.align_hidden_bytes(w, n)
    R = max(4, -(-(1 << 30) // int(nbytes)) + 1)
    hs = [torch.randn(B, T, d, device=dev).to(w.torch_dtype) for _ in range(R)]
    hd = [torch.randn(B, T, d, device=dev).to(w.torch_dtype) for _ in range(R)]
    acc = torch.zeros(1, dtype=torch.float64, device=dev)
    aws = torch.empty(P.align_workspace_size(n), dtype=torch.uint8, device=dev)
    fn = lambda i: P.align_hidden(hs[i], hd[i], acc, workspace=aws)
    res = {"bytes_per_call": nbytes}
    for mode in ("cold", "hot"):
        fn(0)
        us = _timed(fn, 3 * R, (lambda i: i % R) if mode == "cold" else (lambda i: 0))
        res[mode] = {"us": us, "GB/s": nbytes / (us * 1e-6) / 1e9, "frac_of_hbm_peak": nbytes / (us * 1e-6) / 1e9 / PEAK_HBM_GBS}
    out["align_hidden"] = res
    del hs, hd
    # Eq. 10 over B*T rows of the family's vocabulary (each call streams far more than the MALL)
    V = VOCAB[w.block]
    ld = torch.randn(n, V, device=dev).mul_(3.0).to(w.torch_dtype)
    ls = (ld.float() + torch.randn(n, V, device=dev).mul_(0.5)).to(w.torch_dtype)
    kws = torch.empty(P.align_workspace_size(n), dtype=torch.uint8, device=dev)
    fn = lambda i: P.kl_align(ld, ls, acc, workspace=kws)
    nbytes = C.kl_align_bytes(eb, n, V)
    fn(0)
    us = _timed(fn, 3, lambda i: 0)
    out["kl_align"] = {"rows": n, "classes": V, "bytes_per_call": nbytes, "us": us,
                       "GB/s": nbytes / (us * 1e-6) / 1e9, "frac_of_hbm_peak": nbytes / (us * 1e-6) / 1e9 / PEAK_HBM_GBS}
    del ld, ls
    torch.cuda.empty_cache()
    return out


def decode_leg(P, C, w, ks, dev, desc, weights, x0, steps):
    """Incremental decoding (the paper treats prefill only): the stack is
    prefilled over the batch's T tokens into per-layer caches of the kept
    tokens' keys and values, with thresholds = the lowest kept score of each
    (layer, sequence); then decode steps of one new synthetic token per
    sequence, routed by those thresholds on the device. Bytes per step: every
    layer's weights once plus the cached keys and values the step reads."""
    import torch
    B, T, L = w.batch, w.seq, w.n_layers
    dcode = P.F32 if w.dtype == "f32" else P.BF16
    warm = 3
    n = warm + steps
    cap = T + n + steps + 1  # eager steps, then as many replays of a captured step
    ck = [torch.empty(B, w.n_kv_heads, cap, w.head_dim, dtype=w.torch_dtype, device=dev) for _ in range(L)]
    cv = [torch.empty(B, w.n_kv_heads, cap, w.head_dim, dtype=w.torch_dtype, device=dev) for _ in range(L)]
    clen = torch.zeros(L, B, dtype=torch.int32, device=dev)
    thr = torch.empty(L, B, dtype=torch.float32, device=dev)
    x = x0.clone()
    wsp = torch.empty(P.workspace_size(desc, dcode, B, T, max(ks)), dtype=torch.uint8, device=dev)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    P.stack_prefill(desc, weights, ks, x, ck, cv, clen, wsp, thr_out=thr)
    torch.cuda.synchronize()
    prefill_ms = (time.perf_counter() - t0) * 1e3
    del wsp
    lens0 = clen.cpu().numpy()
    ws = torch.empty(P.decode_workspace_size(desc, dcode, B, cap, cap), dtype=torch.uint8, device=dev)
    g = torch.Generator().manual_seed(1234)
    toks = [(torch.randn(B, w.d_model, generator=g) * 0.02).to(w.torch_dtype).to(dev) for _ in range(n)]
    pos = [torch.full((B,), T + i, dtype=torch.int32, device=dev) for i in range(n)]
    keep = torch.zeros(n, L, B, dtype=torch.int32, device=dev)
    for i in range(warm):
        P.decode_step(desc, weights, toks[i], pos[i], cap, thr, ck, cv, clen, ws, keep_out=keep[i])
    lens_start = clen.cpu().numpy()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record()
    for i in range(warm, n):
        P.decode_step(desc, weights, toks[i], pos[i], cap, thr, ck, cv, clen, ws, keep_out=keep[i])
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / steps
    lens_end = clen.cpu().numpy()
    mean_lens = ((lens_start + lens_end) / 2.0).tolist()
    nbytes = C.decode_step_bytes(w, B, mean_lens)
    gbs = nbytes / (ms * 1e-3) / 1e9
    kept = keep[warm:].float().mean().item()
    # the same step captured into a HIP graph and replayed, the next token
    # and its position copied into the captured buffers before each replay
    xg, posg, keepg = toks[0].clone(), pos[0].clone(), torch.zeros(L, B, dtype=torch.int32, device=dev)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        P.decode_step(desc, weights, xg, posg, cap, thr, ck, cv, clen, ws, keep_out=keepg)
    torch.cuda.synchronize()
    e0.record()
    for i in range(steps):
        xg.copy_(toks[i % n])
        posg.fill_(T + n + i)
        graph.replay()
    e1.record()
    torch.cuda.synchronize()
    ms_graph = e0.elapsed_time(e1) / steps
    del graph
    del ck, cv, toks, ws
    torch.cuda.empty_cache()
    return {"tokens_per_s": B / (ms / 1e3), "ms_per_step": ms, "batch": B, "prefill_tokens": T,
            "graph": {"ms_per_step": ms_graph, "tokens_per_s": B / (ms_graph / 1e3),
                      "note": "one captured decode step replayed; each replay preceded by two small copies"},
            "prefill_ms": prefill_ms, "steps": steps, "cache_capacity": cap,
            "cache_len_after_prefill_mean": float(lens0.mean()), "kept_fraction_decode": kept,
            "roofline": {"bound": "hbm", "bytes_per_step": nbytes, "achieved": gbs, "peak": PEAK_HBM_GBS,
                         "unit": "GB/s", "frac": gbs / PEAK_HBM_GBS},
            "note": "routing rule at decode time (not in the paper): keep iff score >= the prefill's lowest kept "
                    "score of that (layer, sequence)"}




def layer_backward_leg(P, C, S, w, ks, dev, desc, weights, x0, reps=10):
    """The routed layer's backward (training side of Section 3.4) at layer 0's
    shape: dsf_sparse_block_backward (activations recomputed from the layer
    input, block adjoint, every weight gradient) against the layer's forward.
    The work of the backward is the recomputed forward plus about twice its
    projection and attention FLOPs."""
    import torch
    B, T, d = w.batch, w.seq, w.d_model
    k = ks[0]
    dl = P.DeviceLayer(S.layer_weights(w, 0), dev)
    g = torch.Generator().manual_seed(5)
    dy = (torch.randn(B, T, d, generator=g) * 0.02).to(w.torch_dtype).to(dev)
    idx = torch.stack([torch.sort(torch.randperm(T, generator=g)[:k])[0] for _ in range(B)]).to(torch.int32).to(dev)
    dx = torch.empty_like(x0)
    shapes = {"w_qkv": (w.d_qkv, d), "b_qkv": (w.d_qkv,), "w_o": (d, w.d_attn), "w_up": (w.d_up, d),
              "w_down": (d, w.d_ff), "norm1_w": (d,), "norm2_w": (d,)}
    if w.block == S.NEOX:
        shapes.update(b_o=(d,), b_up=(w.d_ff,), b_down=(d,), norm1_b=(d,), norm2_b=(d,))
    grads = {n: torch.empty(sh, device=dev) for n, sh in shapes.items()}
    ws = torch.empty(P.backward_workspace_size(desc, P.BF16, B, T, k), dtype=torch.uint8, device=dev)
    wsf = torch.empty(P.workspace_size(desc, P.BF16, B, T, k), dtype=torch.uint8, device=dev)
    fn = lambda: P.sparse_block_backward(desc, dl.weights, x0, dy, idx, dx, grads, ws)
    fwd = lambda xx: P.sparse_block_forward(desc, dl.weights, xx, k, wsf, idx_in=idx)
    fn()
    xs = [x0.clone() for _ in range(reps)]
    fwd(xs[0])
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for i in range(reps):
        fwd(xs[i])
    e1.record()
    torch.cuda.synchronize()
    fwd_ms = e0.elapsed_time(e1) / reps
    e0.record()
    for _ in range(reps):
        fn()
    e1.record()
    torch.cuda.synchronize()
    bwd_ms = e0.elapsed_time(e1) / reps
    fl = C.proj_flops(w, B, k) + C.attn_flops(w, B, k)
    del ws, wsf, xs, grads
    torch.cuda.empty_cache()
    return {"k": k, "forward_ms": fwd_ms, "backward_ms": bwd_ms, "backward_over_forward": bwd_ms / fwd_ms,
            "backward_tflops": 3.0 * fl / (bwd_ms / 1e3) / 1e12,
            "note": "backward recomputes the kept rows' activations (one forward of the block) and computes the "
                    "adjoint (about twice the forward's projection and attention FLOPs); work counted as 3x the "
                    "block's forward FLOPs"}


KIND_DESC = {
    "gemm_qkv": "QKV projection with bias and RoPE at the kept tokens' positions (EPI_QKV_ROPE epilogue)",
    "gemm_o": "attention-output projection with the residual add (EPI_RESID_STORE epilogue)",
    "gemm_up": "FFN up projection: gate|up with SwiGLU (Qwen) or up with bias and GELU (NeoX)",
    "gemm_down": "last projection of the layer with the residual scatter (NeoX fuses W_o and W_down along K)",
    "attn": "causal attention over the kept tokens",
    "router": "router + per-sequence Top-K (one launch)",
    "norm": "gather of the kept rows + normalisation",
}


def cpu_baseline_slice(w, ks, layer, min_seconds=8.0):
    """The oracle, as it stands, on one layer of one sequence at the full
    shape (router over all T tokens, Top-K, the block on the k_l kept rows,
    the scatter), extrapolated to the whole stack over the whole batch with
    the analytic FLOP model (costs.stack_flops over costs.layer_flops of the
    slice). Sequences are run until `min_seconds` have elapsed (at least one).
    """
    from threadpoolctl import threadpool_info

    import synthetic as S
    from oracle import adadsf_oracle as O
    from paper_2607_21291_amd import costs as C

    desc = dict(block=w.block, n_heads=w.n_heads, n_kv_heads=w.n_kv_heads, head_dim=w.head_dim, d_ff=w.d_ff,
                rotary_dims=w.rotary_dims, rope_theta=w.rope_theta, norm_eps=w.norm_eps)
    W = {k: (O.f64(v) if hasattr(v, "detach") else v) for k, v in S.layer_weights(w, layer).items()}
    xall = S.hidden_states(w)
    k = ks[layer]
    dt, nseq = 0.0, 0
    while nseq < w.batch and (nseq == 0 or dt < min_seconds):
        x = O.f64(xall[nseq:nseq + 1])
        t0 = time.perf_counter()
        O.routed_layer(desc, W, x, k)
        dt += time.perf_counter() - t0
        nseq += 1
    threads = max([i.get("num_threads", 1) for i in threadpool_info()] + [1])
    slice_flops = nseq * C.layer_flops(w, 1, w.seq, k, True)
    stack_flops = C.stack_flops(w, w.batch, w.seq, ks, True)
    gflops = slice_flops / dt / 1e9
    tokens_per_s = w.batch * w.seq / (stack_flops / (slice_flops / dt))
    return {"value": tokens_per_s, "unit": "tokens/s", "cores": threads, "kind": "oracle",
            "sample": f"layer {layer} (k={k}) of {w.n_layers}, sequences 0..{nseq - 1} of {w.batch} at T={w.seq}: "
                      f"{dt:.1f} s for {slice_flops / 1e12:.2f} TFLOP ({gflops:.0f} GFLOP/s in fp64); "
                      f"extrapolated to the {w.n_layers}-layer stack over {w.batch} sequences by the analytic "
                      f"FLOP model ({stack_flops / 1e12:.1f} TFLOP per step)",
            "extrapolated": True, "seconds": dt, "gflops": gflops, "cpu_count": os.cpu_count()}


def device_stack(P, S, w, dev):
    layers = [P.DeviceLayer(S.layer_weights(w, l), dev) for l in range(w.n_layers)]
    return layers, [dl.weights for dl in layers]


def calibrate(P, C, w, dev, desc, dcode, weights, x0):
    """Dense calibration pass with the on-GPU similarity statistic (Eq. 4):
    returns (s per layer, wall ms of one pass, rate of the statistic's kernels)."""
    import torch
    B, T, L = w.batch, w.seq, w.n_layers
    ws_cal = torch.empty(P.workspace_size(desc, dcode, B, T, T, True), dtype=torch.uint8, device=dev)
    accum = torch.zeros(L, 2, dtype=torch.float64, device=dev)
    xc = x0.clone()
    P.stack_forward(desc, weights, [T] * L, xc, ws_cal, flags=P.FLAG_DENSE, sim_accum=accum)  # warm
    accum.zero_()
    xc.copy_(x0)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    P.stack_forward(desc, weights, [T] * L, xc, ws_cal, flags=P.FLAG_DENSE, sim_accum=accum)
    s_meas = P.sim_finalize(accum)
    t_cal = time.perf_counter() - t0
    P.timing_enable(4 * L + 8, ["sim"])
    accum.zero_()
    xc.copy_(x0)
    P.stack_forward(desc, weights, [T] * L, xc, ws_cal, flags=P.FLAG_DENSE, sim_accum=accum)
    torch.cuda.synchronize()
    n_sim, ms_sim = P.timing_read("sim")
    P.timing_enable(0)
    sim_rate = {"ms_per_layer": ms_sim / max(n_sim, 1), "launches": n_sim,
                "achieved": C.sim_bytes(w, B, T) * n_sim / (ms_sim / 1e3) / 1e9 if ms_sim > 0 else None,
                "unit": "GB/s", "peak": PEAK_HBM_GBS}
    if sim_rate["achieved"]:
        sim_rate["frac"] = sim_rate["achieved"] / PEAK_HBM_GBS
    del ws_cal, xc
    return s_meas, t_cal * 1e3, sim_rate


def timed_steps(P, desc, weights, ks, x0, ws, steps, warmup, flags=0, dom_kind=None, L=None):
    """Wall ms per step over `steps` stack calls (pristine input copies made
    beforehand), the per-step event times, and (dom_kind given) the launches
    of that kernel kind bracketed by HIP events: (launches, total ms)."""
    import torch
    stream = torch.cuda.current_stream()
    xs = [x0.clone() for _ in range(steps)]
    xw = x0.clone()
    for _ in range(warmup):
        xw.copy_(x0)
        P.stack_forward(desc, weights, ks, xw, ws, flags=flags)
    torch.cuda.synchronize()
    if dom_kind:
        P.timing_enable(steps * len(ks) * 2 + 8, [dom_kind])
    marks = [torch.cuda.Event(enable_timing=True) for _ in range(steps + 1)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(steps):
        marks[i].record(stream)
        P.stack_forward(desc, weights, ks, xs[i], ws, flags=flags)
    marks[-1].record(stream)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    dom = (0, 0.0)
    if dom_kind:
        dom = P.timing_read(dom_kind)
        P.timing_enable(0)
    status = P.workspace_status(ws)
    if status:
        raise RuntimeError(f"workspace status {status:#x} after the timed steps (a stream-K wait gave up)")
    per_step = sorted(marks[i].elapsed_time(marks[i + 1]) for i in range(steps))
    del xs, xw
    return elapsed * 1e3 / steps, per_step, dom


def breakdown_pass(P, C, w, desc, weights, ks, x0, ws, nb):
    """Every launch bracketed by events (a separate pass): ms per step of each
    kernel kind and its rate against its own roofline."""
    import torch
    B, T, L = w.batch, w.seq, w.n_layers
    xw = x0.clone()
    P.timing_enable(nb * L * 16 + 64)
    for i in range(nb):
        xw.copy_(x0)
        P.stack_forward(desc, weights, ks, xw, ws)
    torch.cuda.synchronize()
    out = {}
    for kind in P.KINDS:
        n, ms = P.timing_read(kind)
        if n:
            out[kind] = {"ms_per_step": ms / nb, "launches_per_step": n / nb}
    P.timing_enable(0)
    for kind, v in out.items():
        wk = [C.kind_work(w, kind, B, T, k) for k in ks if k > 0]
        if not wk or wk[0] is None:
            continue
        total, unit = sum(x[0] for x in wk), wk[0][1]
        secs = v["ms_per_step"] / 1e3
        if unit == "flop":
            v.update(achieved=total / secs / 1e12, unit="TFLOP/s", peak=PEAK_BF16_TFLOPS,
                     frac=total / secs / 1e12 / PEAK_BF16_TFLOPS)
        else:
            v.update(achieved=total / secs / 1e9, unit="GB/s", peak=PEAK_HBM_GBS,
                     frac=total / secs / 1e9 / PEAK_HBM_GBS)
    del xw
    return out


def measure_stack(P, C, S, w, dev, steps, warmup, dense=True, breakdown=True, calib=True, only_sparse=False):
    """One workload: retention (fixed, from its similarity profile, or from
    the GPU calibration pass), the timed sparse stack with its dominant
    kernel's roofline, the per-kind breakdown, and the dense stack with the
    same kernels."""
    import torch
    B, T, L = w.batch, w.seq, w.n_layers
    dcode = P.F32 if w.dtype == "f32" else P.BF16
    desc = P.make_desc(w.block, w.d_model, w.n_heads, w.n_kv_heads, w.head_dim, w.d_ff, w.rotary_dims,
                       w.d_router, w.norm_eps, w.rope_theta)
    log(f"workload {w.name}: L={L} d={w.d_model} B={B} T={T} dtype={w.dtype}")
    layers, weights = device_stack(P, S, w, dev)
    x0 = S.hidden_states(w).to(dev)
    s_meas, t_cal, sim_rate = None, None, None
    if w.retention is None and (w.similarity is None or (calib and not only_sparse)):
        s_meas, t_cal, sim_rate = calibrate(P, C, w, dev, desc, dcode, weights, x0)
        log(f"calibration pass {t_cal:.2f} ms; measured similarity {[round(v, 4) for v in s_meas]}")
    r = retention(P, w, s_meas)
    ks = [P.k_from_retention(v, T) for v in r]
    log(f"k per layer {ks}")
    ws = torch.empty(P.workspace_size(desc, dcode, B, T, max(ks)), dtype=torch.uint8, device=dev)

    breakdown_d = {}
    dom_kind = "gemm_up" if only_sparse else None
    if breakdown and not only_sparse:
        breakdown_d = breakdown_pass(P, C, w, desc, weights, ks, x0, ws, min(steps, 5))
        dom_kind = max(breakdown_d, key=lambda kk: breakdown_d[kk]["ms_per_step"])
    breakdown_1s = None
    if breakdown and not only_sparse and w.block == S.NEOX:
        # the NeoX up projection shares the chip with QKV and attention on the
        # second stream, so the in-stack rates above include each other's
        # share; the same pass on one stream gives each kind alone
        prev = os.environ.get("DSF_SINGLE_STREAM")
        os.environ["DSF_SINGLE_STREAM"] = "1"
        try:
            breakdown_1s = breakdown_pass(P, C, w, desc, weights, ks, x0, ws, min(steps, 5))
        finally:
            if prev is None:
                del os.environ["DSF_SINGLE_STREAM"]
            else:
                os.environ["DSF_SINGLE_STREAM"] = prev
    ms_step, per_step, (n_dom, ms_dom) = timed_steps(P, desc, weights, ks, x0, ws, steps, warmup, dom_kind=dom_kind)
    tokens_per_s = B * T / (ms_step / 1e3)
    log(f"sparse stack {ms_step:.3f} ms/step, {tokens_per_s / 1e6:.4f} M tokens/s")

    roofline = None
    if dom_kind and n_dom:
        work = [C.kind_work(w, dom_kind, B, T, k) for k in ks if k > 0]
        total = sum(x[0] for x in work) * steps
        unit = work[0][1]
        launches_expected = len(work) * steps
        per_launch = total / max(n_dom, 1)
        if unit == "flop":
            achieved = total / (ms_dom / 1e3) / 1e12
            roofline = {"bound": "mfma", "achieved": achieved, "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s",
                        "frac": achieved / PEAK_BF16_TFLOPS}
        else:
            achieved = total / (ms_dom / 1e3) / 1e9
            roofline = {"bound": "hbm", "achieved": achieved, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                        "frac": achieved / PEAK_HBM_GBS}
        roofline.update(traffic=measured_traffic(w.name, dom_kind), kernel_kind=dom_kind,
                        kernel=KIND_DESC.get(dom_kind, dom_kind), launches=n_dom,
                        launches_expected=launches_expected, avg_launch_us=ms_dom / max(n_dom, 1) * 1e3,
                        work_per_launch=per_launch, work_unit=unit,
                        share_of_gpu_time=(breakdown_d[dom_kind]["ms_per_step"] /
                                           sum(v["ms_per_step"] for v in breakdown_d.values()))
                        if breakdown_d else None)

    gemm_ms = sum(v["ms_per_step"] for kk, v in breakdown_d.items() if kk.startswith("gemm"))
    rates = {
        "step_tflops": C.stack_flops(w, B, T, ks, True) / (ms_step / 1e3) / 1e12,
        "gemm_tflops": sum(C.proj_flops(w, B, k) for k in ks) / (gemm_ms / 1e3) / 1e12 if gemm_ms else None,
    }
    res = {"workload": w.name, "ms_per_step": ms_step, "ms_per_step_median": per_step[len(per_step) // 2],
           "ms_per_step_min": per_step[0], "tokens_per_s": tokens_per_s, "k_per_layer": ks,
           "mean_retention": sum(r) / L, "roofline": roofline, "kernel_breakdown": breakdown_d, "rates": rates,
           "calibration_ms": t_cal, "similarity_kernel": sim_rate, "similarity_measured": s_meas,
           "flop_ratio_sparse_over_dense": C.stack_flops(w, B, T, ks, True) / C.stack_flops(w, B, T, [T] * L, False)}
    if breakdown_1s is not None:
        res["kernel_breakdown_one_stream"] = breakdown_1s
    if dense and not only_sparse:
        wsd = torch.empty(P.workspace_size(desc, dcode, B, T, T), dtype=torch.uint8, device=dev)
        nd = max(3, steps // 4)
        dense_ms, _, _ = timed_steps(P, desc, weights, [T] * L, x0, wsd, nd, 1, flags=P.FLAG_DENSE)
        res["dense"] = {"ms_per_step": dense_ms, "speedup_sparse_vs_dense": dense_ms / ms_step,
                        "ideal_speedup": 1.0 / res["flop_ratio_sparse_over_dense"]}
        log(f"dense stack {dense_ms:.3f} ms/step, speedup {dense_ms / ms_step:.2f}x "
            f"(1/FLOP ratio {1.0 / res['flop_ratio_sparse_over_dense']:.2f}x)")
        del wsd
    ctx = {"desc": desc, "weights": weights, "layers": layers, "x0": x0, "ws": ws, "ks": ks}
    return res, ctx


def retention_sweep(P, C, S, w, dev, rs, steps, warmup):
    """Uniform retention r for every layer, each r against the dense stack
    (same kernels, same weights): ms/step, speedup and the FLOP ratio."""
    import torch
    B, T, L = w.batch, w.seq, w.n_layers
    dcode = P.F32 if w.dtype == "f32" else P.BF16
    desc = P.make_desc(w.block, w.d_model, w.n_heads, w.n_kv_heads, w.head_dim, w.d_ff, w.rotary_dims,
                       w.d_router, w.norm_eps, w.rope_theta)
    log(f"retention sweep {w.name}: L={L} d={w.d_model} B={B} T={T}, r in {rs}")
    layers, weights = device_stack(P, S, w, dev)
    x0 = S.hidden_states(w).to(dev)
    wsd = torch.empty(P.workspace_size(desc, dcode, B, T, T), dtype=torch.uint8, device=dev)
    dense_ms, _, _ = timed_steps(P, desc, weights, [T] * L, x0, wsd, steps, warmup, flags=P.FLAG_DENSE)
    out = {"workload": f"{w.name}: {L} x {w.d_model}, heads {w.n_heads}/{w.n_kv_heads} x {w.head_dim}, "
                       f"FFN {w.d_ff}, batch {B} x seq {T}", "dense_ms_per_step": dense_ms, "r": {}}
    for r in rs:
        ks = [P.k_from_retention(r, T)] * L
        ms, _, _ = timed_steps(P, desc, weights, ks, x0, wsd, steps, warmup)
        ratio = C.stack_flops(w, B, T, ks, True) / C.stack_flops(w, B, T, [T] * L, False)
        out["r"][f"{r:g}"] = {"k": ks[0], "ms_per_step": ms, "tokens_per_s": B * T / (ms / 1e3),
                              "speedup_vs_dense": dense_ms / ms, "flop_ratio": ratio, "ideal_speedup": 1.0 / ratio}
        log(f"  r={r:g}: {ms:.3f} ms/step, {dense_ms / ms:.2f}x dense (1/FLOP ratio {1.0 / ratio:.2f}x)")
    del layers, weights, x0, wsd
    torch.cuda.empty_cache()
    return out


def main():
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="qwen7b")
    ap.add_argument("--retention", type=float, default=None,
                    help="uniform retention r for every layer (skips the allocation and the calibration pass)")
    ap.add_argument("--batch", type=int, default=None, help="override the workload's batch")
    ap.add_argument("--seq", type=int, default=None, help="override the workload's sequence length")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-dense", action="store_true", help="skip the dense-stack comparison run")
    ap.add_argument("--no-extras", action="store_true",
                    help="skip the other workloads and the standalone sections (used for the counter passes)")
    ap.add_argument("--only-sparse", action="store_true",
                    help="launch only the sparse stack (calibration if the workload needs it, warmup, timed "
                         "steps with the gate/up projection's launches timed): no dense run, no breakdown pass, "
                         "no CPU baseline, no extras; used under rocprofv3")
    args = ap.parse_args()
    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print("bench.py measures one GPU only: the depth-sparse stack is data-parallel over sequences with no "
              "exchange in the forward pass, so this build runs and reports the single-GPU shard "
              "(--gpus 1).", file=sys.stderr)
        sys.exit(2)

    import torch

    import paper_2607_21291_amd as P
    import synthetic as S
    from paper_2607_21291_amd import costs as C

    dev = torch.device("cuda:0")
    w = S.WORKLOADS[args.workload]
    if args.batch or args.seq:
        w = w.replace(batch=args.batch or w.batch, seq=args.seq or w.seq)
        w = w.replace(name=f"{w.name}_B{w.batch}_T{w.seq}")
    if args.retention is not None:
        if not 0.0 < args.retention <= 1.0:
            ap.error("--retention must be in (0, 1]")
        w = w.replace(name=f"{w.name}_r{args.retention:g}", retention=(args.retention,) * w.n_layers,
                      similarity=None)
    if args.only_sparse:
        args.no_dense = args.no_cpu_baseline = args.no_extras = True

    head, ctx = measure_stack(P, C, S, w, dev, args.steps, args.warmup, dense=not args.no_dense,
                              only_sparse=args.only_sparse)
    B, T, L = w.batch, w.seq, w.n_layers
    ks = head["k_per_layer"]
    out = {
        "metric": METRIC,
        "value": head["tokens_per_s"],
        "unit": "tokens/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": head["ms_per_step"],
        "ms_per_step_median": head["ms_per_step_median"],
        "ms_per_step_min": head["ms_per_step_min"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": w.dtype,
        "data": "synthetic (seeded N(0, 0.02) hidden states and random-init weights of the stated shape)",
        "config": {"workload": f"{w.name}: {L}-layer {w.block} stack, d={w.d_model}, heads {w.n_heads}/{w.n_kv_heads}"
                               f"x{w.head_dim}, FFN {w.d_ff}, batch {B} x seq {T}",
                   "global_batch": B, "seq_len": T, "layers": L, "parallelism": "single GPU",
                   "mean_retention": head["mean_retention"], "k_per_layer": ks},
        "roofline": head["roofline"],
        "cpu_baseline": None,
        "kernel_breakdown": head["kernel_breakdown"],
        "rates": head["rates"],
        "dense": head.get("dense"),
        "flop_ratio_sparse_over_dense": head["flop_ratio_sparse_over_dense"],
        "calibration_ms": head["calibration_ms"],
        "similarity_kernel": head["similarity_kernel"],
        "similarity_measured": head["similarity_measured"],
        "hip_runtime": torch.version.hip,
    }
    del ctx
    torch.cuda.empty_cache()
    if not args.no_extras:
        extras = {}
        # GPT-NeoX-160M shape (similarity profile) with the standalone sections
        w2 = S.WORKLOADS["neox160m"]
        r2, c2 = measure_stack(P, C, S, w2, dev, 20, 5)
        kmean = int(round(sum(r2["k_per_layer"]) / len(r2["k_per_layer"])))
        log(f"streaming entry points standalone (neox160m, k={kmean}), cold and hot inputs")
        r2["streaming_kernels"] = streaming_rates(P, C, w2, kmean, dev, S.layer_weights(w2, 0))
        log("router-score pathway: gated stack, gate score gradient, router backward")
        r2["router_score_pathway"] = router_pathway(P, C, w2, c2["ks"], dev, c2["desc"], c2["weights"], c2["x0"],
                                                    c2["ws"], r2["ms_per_step"], 6, S.layer_weights(w2, 0))
        log("alignment objective: teacher/student stack, Eq. 9 and Eq. 10 kernels")
        r2["alignment_objective"] = alignment_objective(P, C, w2, c2["ks"], dev, c2["desc"], c2["weights"], c2["x0"],
                                                        r2["ms_per_step"], 6)
        log("routed layer backward at layer 0's shape")
        r2["layer_backward"] = layer_backward_leg(P, C, S, w2, c2["ks"], dev, c2["desc"], c2["weights"], c2["x0"])
        log("incremental decoding: prefill into kept-token caches, then threshold-routed decode steps")
        r2["decode"] = decode_leg(P, C, w2, c2["ks"], dev, c2["desc"], c2["weights"], c2["x0"], 20)
        extras["neox160m"] = r2
        del c2
        torch.cuda.empty_cache()
        # Qwen2.5-0.5B shape, similarity profile
        r3, c3 = measure_stack(P, C, S, S.WORKLOADS["qwen05b"], dev, 10, 3)
        extras["qwen05b"] = r3
        del c3
        torch.cuda.empty_cache()
        # GPT-NeoX-1.4B shape, uniform retention sweep
        extras["neox14b_sweep"] = retention_sweep(P, C, S, S.WORKLOADS["neox14b"], dev, [1.0, 0.75, 0.5, 0.25], 5, 2)
        # the paper's evaluation shapes at its retention ratios (Tables 1b, 2)
        paper = {}
        for name, seq in (("neox130m", None), ("qwen05b", 2048), ("qwen15b", None)):
            wp = S.WORKLOADS[name]
            if seq:
                wp = wp.replace(name=f"{name}_T{seq}", seq=seq, similarity=None, target=None, tau=None,
                                retention=(0.8,) * wp.n_layers)
            paper[wp.name] = retention_sweep(P, C, S, wp, dev, [0.9, 0.8, 0.7], 5, 2)
        extras["paper_shapes"] = paper
        out["extras"] = extras
    if not args.no_cpu_baseline:
        layer = min(range(L), key=lambda l: abs(ks[l] - sorted(ks)[L // 2]))
        log(f"cpu oracle baseline: layer {layer} of one sequence at full shape, extrapolated")
        out["cpu_baseline"] = cpu_baseline_slice(w, ks, layer)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
