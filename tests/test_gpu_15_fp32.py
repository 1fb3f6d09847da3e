"""fp32 on the fp32 matrix cores: routed layers whose projections take each of
the row-tile sizes (and the scalar kernel, for reductions that are no multiple
of 16), attention lengths around the 16-query and 32-key blocks, infinite
values that only later queries may see, and the router's 16-token blocks,
against the oracle. Tolerances: gpu_util.TOL for layers; attention and router
within fp32 accumulation bounds of the float64 result."""
import numpy as np
import pytest
import torch

import paper_2607_21291_amd as P
import synthetic as S
from oracle import adadsf_oracle as O

from gpu_util import U32, announce, check_layer, router_bound, run_layer, to_np

pytestmark = pytest.mark.gpu


def _w(block, d, hq, hkv, hd, f, rot, B, T):
    base = S.WORKLOADS["tiny_neox_f32" if block == S.NEOX else "tiny_qwen_f32"]
    return base.replace(name="fp32", d_model=d, n_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=f, rotary_dims=rot, batch=B,
                        seq=T)


LAYERS = [
    (S.NEOX, 256, 4, 4, 64, 1024, 16, 1, 80, 65),    # one row past a tile of 64
    (S.NEOX, 256, 4, 4, 64, 1024, 16, 3, 170, 150),
    (S.NEOX, 256, 4, 4, 64, 1024, 16, 8, 300, 300),  # 2400 rows: tiles of 64 x 64
    (S.QWEN, 256, 6, 2, 64, 512, 64, 2, 100, 77),
    (S.QWEN, 384, 3, 1, 128, 640, 128, 2, 120, 97),
    (S.QWEN, 264, 8, 2, 32, 512, 32, 2, 90, 81),     # d = 264: scalar kernel where it is the reduction
    (S.NEOX, 128, 4, 4, 32, 512, 8, 2, 90, 81),      # rotation halves of 4: scalar QKV
]


@pytest.mark.parametrize("flags", [0, P.FLAG_GATE])
@pytest.mark.parametrize("case", LAYERS, ids=lambda c: f"{c[0]}-d{c[1]}-h{c[2]}.{c[3]}x{c[4]}-B{c[7]}-k{c[9]}")
def test_layer(dev, case, flags):
    *shape, k = case
    w = _w(*shape)
    W = S.layer_weights(w, 0)
    x = S.hidden_states(w)
    announce(f"fp32 layer {case} flags={flags}")
    y, scores, idx = run_layer(dev, w, W, x, k, flags=flags)
    check_layer(w, W, x, y, scores, idx, k, gate=bool(flags), sample=[0, w.batch - 1])


@pytest.mark.parametrize("hd,hq,hkv", [(32, 2, 2), (64, 4, 2), (128, 3, 1)])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 33, 128, 129, 270])
def test_attention(dev, n, hd, hq, hkv):
    g = torch.Generator().manual_seed(n * 100 + hd)
    q, k, v = (torch.randn(2, h, n, hd, generator=g) * s for h, s in ((hq, 3.0), (hkv, 1.0), (hkv, 1.0)))
    out = torch.empty(2, n, hq * hd, device=dev)
    announce(f"fp32 attention n={n} hd={hd}")
    P.attention_forward(q.to(dev), k.to(dev), v.to(dev), out)
    got = to_np(out).reshape(2, n, hq, hd)
    for b in range(2):
        qf, kf, vf = (to_np(t[b]).transpose(1, 0, 2) for t in (q, k, v))
        ref = O.causal_attention(qf, kf, vf).reshape(n, hq, hd)
        # scores carry |s| (hd + 4) u of error, the weighted mean (n + 8) u of the largest value
        smax = np.max(np.abs(qf)) * np.max(np.abs(kf)) * np.sqrt(hd)
        assert np.max(np.abs(got[b] - ref)) < U32 * (2 * smax * (hd + 4) + n + 8) * np.max(np.abs(vf))


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_attention_future_values_do_not_leak(dev, bad):
    n, hd = 50, 64
    g = torch.Generator().manual_seed(3)
    q, k, v = (torch.randn(1, 2, n, hd, generator=g) for _ in range(3))
    v[0, 0, 37, 5] = bad
    out = torch.empty(1, n, 2 * hd, device=dev)
    announce(f"fp32 attention with {bad} at key 37")
    P.attention_forward(q.to(dev), k.to(dev), v.to(dev), out)
    o = out.cpu().reshape(n, 2, hd)
    hit = torch.zeros(n, 2, hd, dtype=torch.bool)
    hit[37:, 0, 5] = True
    assert torch.isfinite(o[~hit]).all()
    assert not torch.isfinite(o[hit]).any()
    v[0, 0, 37, 5] = 0.0
    ref = torch.empty(1, n, 2 * hd, device=dev)
    P.attention_forward(q.to(dev), k.to(dev), v.to(dev), ref)
    assert torch.equal(o[~hit], ref.cpu().reshape(n, 2, hd)[~hit])


@pytest.mark.parametrize("key", [32, 37, 64])
def test_attention_infinitely_low_scores_weigh_nothing(dev, key):
    # a key whose score is -inf for every query: the first or only visible key
    # of a wave's tile for some of them
    n, hd = 70, 64
    g = torch.Generator().manual_seed(5)
    q, k, v = (torch.randn(1, 1, n, hd, generator=g) for _ in range(3))
    q[..., 0] = q[..., 0].abs() + 0.5
    k[0, 0, key, 0] = -float("inf")
    out = torch.empty(1, n, hd, device=dev)
    announce(f"fp32 attention with scores of -inf at key {key}")
    P.attention_forward(q.to(dev), k.to(dev), v.to(dev), out)
    s = to_np(q[0, 0]) @ to_np(k[0, 0]).T / np.sqrt(hd)
    s[np.triu_indices(n, 1)] = -np.inf
    e = np.exp(s - s.max(1, keepdims=True))
    ref = (e / e.sum(1, keepdims=True)) @ to_np(v[0, 0])
    # the bound of test_attention, with the largest finite score
    smax = np.max(np.abs(s[np.isfinite(s)])) * hd
    assert np.max(np.abs(to_np(out[0]) - ref)) < U32 * (2 * smax * (hd + 4) + n + 8) * np.max(np.abs(to_np(v)))


@pytest.mark.parametrize("d_r", [16, 32, 48, 64])
@pytest.mark.parametrize("n,d", [(1, 128), (16, 136), (17, 768), (100, 8)])
def test_router(dev, n, d, d_r):
    g = torch.Generator().manual_seed(n + d + d_r)
    rn = lambda *s: torch.randn(*s, generator=g)
    W = {"router_w1": rn(d_r, d), "router_b1": rn(d_r), "router_w2": rn(d_r), "router_b2": 0.5}
    x = rn(1, n, d)
    sc = torch.empty(1, n, device=dev)
    announce(f"fp32 router n={n} d={d} d_r={d_r}")
    P.router_score(x.to(dev), W["router_w1"].to(dev), W["router_b1"].to(dev), W["router_w2"].to(dev), 0.5, sc)
    ref = O.router_scores(x, W["router_w1"], W["router_b1"], W["router_w2"], 0.5)
    assert np.all(np.abs(to_np(sc) - ref) <= router_bound(to_np(x), W, "f32"))
