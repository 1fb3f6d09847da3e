"""Weight, bias and norm gradients of the layer's backward at the edges of
their kernels: output tiles of 128 with remainders (d = 136), reductions of
one token, around a tile of 64 tokens and long enough for 2 to 8 token slices
per tile, norm rows of each width class (one wavefront per row up to 2048,
four beyond), and any subset of the gradients. Against the oracle's float64
gradients, 2e-2 of each one's infinity norm as for the layer; a gradient
asked for alone is held to the same bound."""
import numpy as np
import pytest
import torch

import paper_2607_21291_amd as P
import synthetic as S
from oracle import adadsf_oracle as O

from gpu_util import TOL, announce, desc_dict, make_desc, rel_inf, workload
from test_gpu_12_backward import _grads, check_backward, run_backward

pytestmark = pytest.mark.gpu


def _case(block, d, hq, hkv, hd, f, B, T, k):
    base = workload("neox_bf16_small" if block == S.NEOX else "qwen_bf16_small")
    w = base.replace(name="wgrad", d_model=d, n_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=f,
                     rotary_dims=hd if block == S.QWEN else hd // 4, batch=B, seq=T)
    return _inputs(w, k)


def _inputs(w, k):
    W = S.layer_weights(w, 0)
    x = S.hidden_states(w)
    g = torch.Generator().manual_seed(w.d_model + k)
    dy = torch.randn(w.batch, w.seq, w.d_model, generator=g).to(torch.bfloat16)
    idx = np.stack([np.sort(torch.randperm(w.seq, generator=g)[:k].numpy()) for _ in range(w.batch)])
    return w, W, x, dy, idx


@pytest.mark.parametrize("case", [
    (S.NEOX, 136, 2, 2, 32, 192, 1, 9, 1),
    (S.NEOX, 136, 3, 3, 64, 192, 1, 70, 63),
    (S.NEOX, 264, 4, 4, 64, 576, 1, 70, 65),
    (S.NEOX, 520, 4, 4, 64, 1088, 2, 300, 257),    # 9 token tiles: two slices
    (S.NEOX, 128, 2, 2, 64, 512, 8, 300, 290),     # 37: eight slices of few tiles
    (S.NEOX, 768, 12, 12, 64, 3072, 2, 300, 290),  # 10 token tiles: two slices
    (S.NEOX, 776, 12, 12, 64, 2944, 8, 300, 290),  # three slices, remainders in both directions
    (S.QWEN, 136, 3, 1, 64, 192, 1, 70, 64),
    (S.QWEN, 1032, 4, 1, 128, 320, 2, 170, 161),
    (S.QWEN, 2056, 2, 1, 64, 128, 1, 40, 33),
    (S.NEOX, 2056, 2, 2, 64, 128, 1, 40, 17),
    (S.QWEN, 4104, 2, 1, 64, 64, 1, 40, 33),
    (S.NEOX, 8192, 2, 2, 64, 64, 1, 40, 16),
    (S.NEOX, 2056, 2, 2, 64, 9152, 1, 140, 129),   # up and down: 324 tiles of 256 with remainders, and bias sums
], ids=lambda c: f"{c[0]}-d{c[1]}-f{c[5]}-B{c[6]}-k{c[8]}")
def test_all_gradients(dev, case):
    w, W, x, dy, idx = _case(*case)
    announce(f"weight gradients {case}")
    dx, g = run_backward(dev, w, W, x, dy, idx, False)
    check_backward(w, W, x, dy, idx, False, dx, g)
    dx2, g2 = run_backward(dev, w, W, x, dy, idx, False)
    assert torch.equal(dx, dx2) and all(torch.equal(g[n], g2[n]) for n in g)


@pytest.mark.parametrize("block,hkv", [(S.NEOX, 4), (S.QWEN, 2)])
def test_each_gradient_alone(dev, block, hkv):
    w, W, x, dy, idx = _case(block, 264, 4, hkv, 64, 576, 2, 300, 290)
    B, T, _ = x.shape
    k = idx.shape[1]
    ref = O.routed_layer_backward(desc_dict(w), W, x, dy, idx, gate=False)["grads"]
    dl = P.DeviceLayer(W, dev)
    desc = make_desc(w)
    xd, dyd = x.to(dev), dy.to(dev)
    idd = torch.as_tensor(idx, dtype=torch.int32).to(dev)
    ws = torch.empty(P.backward_workspace_size(desc, P.BF16, B, T, k), dtype=torch.uint8, device=dev)
    full, _ = run_backward(dev, w, W, x, dy, idx, False)
    for name, buf in {**_grads(w, dev), None: None}.items():
        announce(f"only {name}")
        dx = torch.full_like(xd, float("nan"))
        P.sparse_block_backward(desc, dl.weights, xd, dyd, idd, dx, {name: buf} if name else {}, ws)
        torch.cuda.synchronize()
        assert torch.equal(dx, full)
        if name:
            assert rel_inf(buf.double().cpu().numpy(), ref[name]) < TOL[w.dtype], name
