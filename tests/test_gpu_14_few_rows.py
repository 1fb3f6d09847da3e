"""Few-row projections and the decode attention at the sizes where they can go
wrong: row blocks of 16 and their remainders, one and two column groups per
workgroup, output widths that are no multiple of 16, reductions that fall back
to the other kernels, query groups of 1 to 20 heads per kv head, cache lengths
around the chunk of 256 keys, empty and full caches. One decode step on random
caches is compared with the oracle's norms, rotation and activations composed
in float64; short routed layers (at most 64 kept rows, the few-row kernel
without split scratch up to 24) with the oracle's layer."""
import numpy as np
import pytest
import torch

import paper_2607_21291_amd as P
import synthetic as S
from oracle import adadsf_oracle as O

from gpu_util import TOL, announce, check_layer, desc_dict, dtype_code, make_desc, rel_inf, run_layer, to_np, workload

pytestmark = pytest.mark.gpu


def _w(block, d, hq, hkv, hd, f, rot, dtype):
    base = S.WORKLOADS["neox160m" if block == S.NEOX else "qwen05b"]
    return base.replace(name="few", n_layers=1, d_model=d, n_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=f,
                        rotary_dims=rot, dtype=dtype, batch=2, seq=64)


def _step_ref(w, W, x, pos, ck, cv, lens, keep):
    """One token per sequence over its cache, in float64."""
    Hq, Hkv, hd, f = w.n_heads, w.n_kv_heads, w.head_dim, w.d_ff
    y = x.copy()
    for b in np.nonzero(keep)[0]:
        row = x[b:b + 1]
        neox = w.block == S.NEOX
        a = O.layer_norm(row, W["norm1_w"], W["norm1_b"], w.norm_eps) if neox else O.rms_norm(row, W["norm1_w"], w.norm_eps)
        qkv = (a @ O.f64(W["w_qkv"]).T + O.f64(W["b_qkv"])).reshape(1, Hq + 2 * Hkv, hd)
        p = pos[b:b + 1]
        q = O.rope(qkv[:, :Hq], p, w.rotary_dims, w.rope_theta)[0]
        k = np.concatenate([ck[b, :, :lens[b]], O.rope(qkv[:, Hq:Hq + Hkv], p, w.rotary_dims, w.rope_theta)[0][:, None]], 1)
        v = np.concatenate([cv[b, :, :lens[b]], qkv[0, Hq + Hkv:][:, None]], 1)
        out = []
        for h in range(Hq):
            s = k[h // (Hq // Hkv)] @ q[h] / np.sqrt(hd)
            e = np.exp(s - s.max())
            out.append(e @ v[h // (Hq // Hkv)] / e.sum())
        ao = np.concatenate(out)[None] @ O.f64(W["w_o"]).T
        if neox:
            m = O.layer_norm(row, W["norm2_w"], W["norm2_b"], w.norm_eps)
            mo = O.gelu(m @ O.f64(W["w_up"]).T + O.f64(W["b_up"])) @ O.f64(W["w_down"]).T + O.f64(W["b_down"])
            ao = ao + O.f64(W["b_o"])
        else:
            gu = O.rms_norm(row + ao, W["norm2_w"], w.norm_eps) @ O.f64(W["w_up"]).T
            mo = (O.silu(gu[:, :f]) * gu[:, f:]) @ O.f64(W["w_down"]).T
        y[b] = (row + ao + mo)[0]
    return y


STEPS = [
    # block, d, Hq, Hkv, hd, f, R, dtype, B, cap
    (S.NEOX, 256, 4, 4, 64, 512, 16, "bf16", 1, 5),
    (S.NEOX, 256, 4, 4, 64, 512, 16, "bf16", 16, 600),
    (S.NEOX, 256, 4, 4, 64, 512, 16, "bf16", 17, 600),
    (S.NEOX, 256, 2, 2, 128, 512, 32, "bf16", 33, 300),
    (S.NEOX, 256, 8, 8, 32, 512, 32, "bf16", 64, 300),
    (S.NEOX, 256, 4, 4, 64, 512, 16, "bf16", 65, 64),    # past the few-row limit
    (S.NEOX, 264, 4, 4, 64, 512, 16, "bf16", 5, 300),    # reduction of 264: other kernels; N = 264
    (S.NEOX, 256, 4, 4, 64, 512, 8, "bf16", 5, 300),     # rotation halves of 4: split-K QKV
    (S.NEOX, 4104, 2, 2, 64, 64, 16, "bf16", 3, 300),    # wider than the in-launch norm
    (S.QWEN, 256, 4, 2, 64, 8192, 64, "bf16", 3, 520),   # two column groups per workgroup, norm inside
    (S.QWEN, 256, 6, 2, 64, 8192, 64, "bf16", 20, 520),  # the same, norm apart, 3 heads per kv head
    (S.QWEN, 256, 14, 2, 64, 512, 64, "bf16", 40, 257),  # 7 heads per kv head
    (S.QWEN, 256, 4, 2, 64, 8192, 64, "bf16", 37, 520),  # down: K split over workgroups, 33-64 rows
    (S.QWEN, 256, 20, 1, 32, 512, 32, "bf16", 2, 257),   # 20 heads: two head blocks
    (S.QWEN, 128, 7, 1, 128, 17408, 128, "bf16", 20, 257),  # gate|up wide enough for the tile grid
    (S.QWEN, 256, 7, 1, 128, 512, 128, "f32", 3, 520),
    (S.QWEN, 128, 20, 1, 32, 256, 32, "f32", 33, 257),
    (S.NEOX, 128, 2, 2, 64, 256, 16, "f32", 17, 520),
    (S.NEOX, 136, 1, 1, 128, 256, 16, "f32", 2, 520),    # reduction of 136
    (S.QWEN, 128, 4, 2, 64, 256, 64, "f32", 2, 257),
]


@pytest.mark.parametrize("case", STEPS, ids=lambda c: f"{c[0]}-d{c[1]}-h{c[2]}.{c[3]}x{c[4]}-f{c[5]}-r{c[6]}-{c[7]}-B{c[8]}")
def test_decode_step_on_random_caches(dev, case):
    block, d, hq, hkv, hd, f, rot, dtype, B, cap = case
    w = _w(block, d, hq, hkv, hd, f, rot, dtype)
    W = S.layer_weights(w, 0)
    dl = P.DeviceLayer(W, dev)
    g = torch.Generator().manual_seed(B * 1000 + d)
    rn = lambda *s, std=0.5: (torch.randn(*s, generator=g) * std).to(w.torch_dtype)
    x, ck, cv = rn(B, d), rn(B, hkv, cap, hd), rn(B, hkv, cap, hd)
    edges = [0, 1, 63, 64, 255, 256, 257, 511, 512, cap - 1, cap]
    lens = np.array([min(edges[(b + B) % len(edges)], cap) for b in range(B)], dtype=np.int32)
    want = np.array([b % 5 != 3 for b in range(B)])
    pos = torch.randint(0, cap + 7, (B,), generator=g, dtype=torch.int32)
    thr = torch.tensor(np.where(want, -np.inf, np.inf)[None], dtype=torch.float32, device=dev)
    xd, ckd, cvd = x.to(dev), ck.to(dev), cv.to(dev)
    clen = torch.tensor(lens[None], device=dev)
    keep = torch.empty(1, B, dtype=torch.int32, device=dev)
    sc = torch.empty(1, B, device=dev)
    ws = torch.empty(P.decode_workspace_size(make_desc(w), dtype_code(w), B, cap + 7, cap), dtype=torch.uint8, device=dev)
    announce(f"few-row decode step {case}")
    P.decode_step(make_desc(w), [dl.weights], xd, pos.to(dev), cap + 7, thr, [ckd], [cvd], clen, ws, scores_out=sc,
                  keep_out=keep)
    torch.cuda.synchronize()
    kept = want & (lens < cap)
    np.testing.assert_array_equal(keep.cpu().numpy()[0], np.where(kept, 1, np.where(want, 2, 0)))
    np.testing.assert_array_equal(clen.cpu().numpy()[0], lens + kept)
    ref_sc = O.router_scores(O.f64(x)[None], W["router_w1"], W["router_b1"], W["router_w2"])[0]
    assert np.max(np.abs(to_np(sc)[0] - ref_sc)) < 1e-5 * max(1.0, np.max(np.abs(ref_sc)))
    ref = _step_ref(w, W, O.f64(x), pos.numpy().astype(np.int64), O.f64(ck), O.f64(cv), lens, kept)
    got = to_np(xd)
    for b in range(B):
        if not kept[b]:
            assert torch.equal(xd[b].cpu(), x[b])
            assert torch.equal(ckd[b].cpu(), ck[b]) and torch.equal(cvd[b].cpu(), cv[b])
        else:  # the other slots are as they were
            m = torch.ones(cap, dtype=torch.bool)
            m[lens[b]] = False
            assert torch.equal(ckd[b].cpu()[:, m], ck[b][:, m]) and torch.equal(cvd[b].cpu()[:, m], cv[b][:, m])
    if kept.any():
        # the update, beyond the roundings of the stored rows: half an ulp (2^-9 of the value in
        # bf16) of the output and, for the sequential block, of h = x + attention between the two
        # halves, which is no larger than |x| + |update|
        upd = np.abs(ref - O.f64(x))[kept]
        half = 2.0 ** -9 if dtype == "bf16" else 2.0 ** -24
        slack = half * np.abs(ref)[kept]
        if block == S.QWEN:
            slack = slack + half * (np.abs(O.f64(x))[kept] + np.max(upd))
        assert np.max(np.abs(got - ref)[kept] - slack) < TOL[dtype] * np.max(upd)


@pytest.mark.parametrize("flags", [0, P.FLAG_GATE])
@pytest.mark.parametrize("name,k", [("neox_bf16_small", 8), ("neox_bf16_small", 12), ("neox_bf16_small", 13),
                                    ("neox_bf16_small", 32), ("qwen_bf16_small", 9),
                                    ("qwen_bf16_small", 12), ("qwen_bf16_hd128", 25), ("qwen_bf16_hd128", 64), ("neox_bf16_hd128", 17), ("tiny_neox_f32", 7),
                                    ("tiny_qwen_f32", 32)])
def test_short_layer_matches_oracle(dev, name, k, flags):
    w = workload(name)
    W = S.layer_weights(w, 0)
    x = S.hidden_states(w)
    announce(f"few-row layer {name} k={k} flags={flags}")
    y, scores, idx = run_layer(dev, w, W, x, k, flags=flags)
    check_layer(w, W, x, y, scores, idx, k, **({"gate": True} if flags else {}))
    y2, _, _ = run_layer(dev, w, W, x, k, flags=flags)
    assert torch.equal(y, y2)


def _decode(dev, w, Ws, x, pos, cap, max_pos, ck, cv, lens, spare=0):
    """One step of len(Ws) layers, every token kept; returns x, caches."""
    L, B = len(Ws), x.shape[0]
    dls = [P.DeviceLayer(W, dev) for W in Ws]
    xd, cks, cvs = x.to(dev), [c.to(dev) for c in ck], [c.to(dev) for c in cv]
    clen = torch.tensor(lens, dtype=torch.int32).repeat(L, 1).to(dev)
    thr = torch.full((L, B), -float("inf"), device=dev)
    size = P.decode_workspace_size(make_desc(w), dtype_code(w), B, max_pos, cap) - spare
    ws = torch.empty(size, dtype=torch.uint8, device=dev)
    P.decode_step(make_desc(w), [d.weights for d in dls], xd, pos.to(dev), max_pos, thr, cks, cvs, clen, ws)
    torch.cuda.synchronize()
    return xd.cpu(), [c.cpu() for c in cks], [c.cpu() for c in cvs]


@pytest.mark.parametrize("block,B", [(S.NEOX, 24), (S.NEOX, 16), (S.QWEN, 24), (S.QWEN, 16)])
@pytest.mark.parametrize("var,val", [("DSF_GEMM_TILE", "small"), ("DSF_GEMM_SCHEDULE", "classic")])
def test_forced_tiles_reach_the_decode_step(dev, monkeypatch, block, B, var, val):
    # a forced tile or schedule takes a step's projections to the tile grids:
    # on empty caches they then give the bits of a prefill of one token, whose
    # projections run there too (in the NeoX block also the layer's output:
    # attention over one token is its value; its reductions are too short to be
    # cut along K, which only the prefill could)
    w = _w(block, 1024, 16, 16 if block == S.NEOX else 4, 64, 512, 16 if block == S.NEOX else 64, "bf16")
    W = S.layer_weights(w, 0)
    g = torch.Generator().manual_seed(B)
    x = (torch.randn(B, 1024, generator=g) * 0.02).to(torch.bfloat16)
    ck = cv = torch.zeros(B, w.n_kv_heads, 4, 64, dtype=torch.bfloat16)
    monkeypatch.setenv(var, val)
    announce(f"decode step and prefill with {var}={val} B={B}")
    y, dk, dv = _decode(dev, w, [W], x, torch.zeros(B, dtype=torch.int32), 4, 4, [ck], [cv], [0] * B)
    xp, pk, pv = x.to(dev).view(B, 1, 1024), ck.to(dev), torch.zeros_like(cv).to(dev)
    clen = torch.zeros(1, B, dtype=torch.int32, device=dev)
    ws = torch.empty(P.workspace_size(make_desc(w), P.BF16, B, 1, 1, False), dtype=torch.uint8, device=dev)
    P.stack_prefill(make_desc(w), [P.DeviceLayer(W, dev).weights], [1], xp, [pk], [pv], clen, ws)
    torch.cuda.synchronize()
    assert torch.equal(dk[0], pk.cpu()) and torch.equal(dv[0], pv.cpu())
    if block == S.NEOX:
        assert torch.equal(y, xp.cpu().view(B, 1024))


@pytest.mark.parametrize("B", [20, 37])
def test_cache_capacity_does_not_change_the_bits(dev, B):
    # the down projection is split along K over workgroups, as far at any capacity
    w = _w(S.QWEN, 512, 8, 2, 64, 8192, 64, "bf16")
    W = S.layer_weights(w, 0)
    g = torch.Generator().manual_seed(B)
    rn = lambda *s: (torch.randn(*s, generator=g) * 0.5).to(torch.bfloat16)
    x, k, v = (rn(B, 512) * 0.04).to(torch.bfloat16), rn(B, 2, 100, 64), rn(B, 2, 100, 64)
    pos, lens = torch.arange(B, dtype=torch.int32), [(7 * b) % 100 for b in range(B)]
    out = []
    for cap in (101, 4000):
        announce(f"decode step B={B} cap={cap}")
        pad = torch.zeros(B, 2, cap - 100, 64, dtype=torch.bfloat16)
        y, _, _ = _decode(dev, w, [W], x, pos, cap, 128, [torch.cat([k, pad], 2)], [torch.cat([v, pad], 2)], lens)
        out.append(y)
    assert torch.equal(out[0], out[1])
    # a workspace without the projections' partial sums (those of the attention stay: one chunk of keys)
    announce(f"decode step B={B} short workspace")
    part = -(-4 * B * w.n_heads * (w.head_dim + 2) // 256) * 256
    pad = torch.zeros(B, 2, 1, 64, dtype=torch.bfloat16)
    args = (dev, w, [W], x, pos, 101, 128, [torch.cat([k, pad], 2)], [torch.cat([v, pad], 2)], lens)
    y, _, _ = _decode(*args, spare=(4 << 20) - part)
    assert rel_inf(to_np(y) - to_np(x), to_np(out[0]) - to_np(x)) < TOL["bf16"]
    with pytest.raises(RuntimeError, match="workspace"):
        _decode(*args, spare=(4 << 20) - part + 256)


@pytest.mark.parametrize("B", [20, 37])
def test_split_projections_leave_their_counters_clear(dev, B):
    # two layers in one step, whose launches share the split's counters, give
    # the bits of one layer after the other
    w = _w(S.QWEN, 256, 4, 2, 64, 8192, 64, "bf16")
    Ws = [S.layer_weights(w, l) for l in range(2)]
    cap, g = 300, torch.Generator().manual_seed(B)
    rn = lambda *s: (torch.randn(*s, generator=g) * 0.5).to(torch.bfloat16)
    x, ck, cv = rn(B, 256), [rn(B, 2, cap, 64) for _ in Ws], [rn(B, 2, cap, 64) for _ in Ws]
    pos, lens = torch.arange(B, dtype=torch.int32), [(37 * b) % cap for b in range(B)]
    announce(f"two-layer decode step B={B}")
    y, _, _ = _decode(dev, w, Ws, x, pos, cap, cap, ck, cv, lens)
    one = x
    for l, W in enumerate(Ws):
        one, _, _ = _decode(dev, w, [W], one, pos, cap, cap, ck[l:l + 1], cv[l:l + 1], lens)
    assert torch.equal(y, one)
