"""Attention's share of the layer's backward where its blocks of 64 and 128
queries (keys) begin and end, for each head dimension and grouping, below and
above the number of workgroups from which a wavefront takes two groups of 16
(512 blocks of 128, counted apart for query heads and for kv heads). All
gradients are held to the oracle's float64 ones, 2e-2 of each one's infinity
norm, and repeated calls are equal."""
import pytest
import torch

import synthetic as S

from gpu_util import announce, workload
from test_gpu_12_backward import check_backward, run_backward
from test_gpu_18_weight_grads import _case, _inputs

pytestmark = pytest.mark.gpu


def _workload_case(name, B, T, k, rot):
    w = workload(name).replace(batch=B, seq=T)
    if rot:
        w = w.replace(rotary_dims=rot)
    return _inputs(w, k)


@pytest.mark.parametrize("rot", [None, 8, 20])
@pytest.mark.parametrize("name,B,T,k", [("neox_bf16_small", 2, 90, 77), ("qwen_bf16_hd128", 1, 140, 130)])
def test_rotary_dims(dev, name, B, T, k, rot):
    # rotated dims in multiples of 16 (None: the workload's), which are turned
    # back eight at a time, and others
    w, W, x, dy, idx = _workload_case(name, B, T, k, rot)
    announce(f"attention backward {name} rotary_dims={w.rotary_dims}")
    dx, g = run_backward(dev, w, W, x, dy, idx, False)
    check_backward(w, W, x, dy, idx, False, dx, g)


@pytest.mark.parametrize("case", [
    (S.NEOX, 128, 2, 2, 32, 128, 1, 70, 63),
    (S.NEOX, 128, 2, 2, 32, 128, 1, 140, 129),
    (S.NEOX, 512, 16, 16, 32, 128, 16, 290, 257),   # 768 blocks: two groups per wave
    (S.NEOX, 512, 8, 8, 64, 128, 16, 520, 511),     # 512: the first grid that takes them
    (S.NEOX, 512, 8, 8, 64, 128, 16, 390, 384),     # 384: one group
    (S.QWEN, 512, 16, 2, 64, 128, 16, 270, 193),    # queries with two groups, keys with one
    (S.QWEN, 256, 14, 2, 64, 128, 2, 130, 65),
    (S.QWEN, 256, 6, 2, 128, 128, 3, 200, 191),
], ids=lambda c: f"{c[0]}-h{c[2]}.{c[3]}x{c[4]}-B{c[6]}-k{c[8]}")
def test_attention_blocks(dev, case):
    w, W, x, dy, idx = _case(*case)
    announce(f"attention backward {case}")
    dx, g = run_backward(dev, w, W, x, dy, idx, False)
    check_backward(w, W, x, dy, idx, False, dx, g)
    dx2, g2 = run_backward(dev, w, W, x, dy, idx, False)
    assert torch.equal(dx, dx2) and all(torch.equal(g[n], g2[n]) for n in g)


def test_infinite_key_of_no_weight_keeps_its_value_gradient(dev):
    # 70 tokens, the block of keys padded to 128 queries. Token 20's key has
    # -inf in dim 63 of head 0, where every query is positive: its score is
    # -inf and its weight zero for all of them, so its value's gradient is
    # zero, also after the padding (zero rows, whose score with it is NaN)
    w, W, x, dy, idx = _case(S.NEOX, 128, 2, 2, 64, 192, 1, 70, 70)
    dq, c, t = w.d_attn, 5, 20
    x[0, t, c] = 100.0                  # normalises to sqrt(d - 1) = 11.3, the others stay below 5
    W["w_qkv"][63] = 0.0
    W["b_qkv"][63] = 2.0 ** -120
    W["w_qkv"][dq + 63] = 0.0
    W["w_qkv"][dq + 63, c] = -3.75e37   # 11.3 times it is beyond the largest bf16
    W["b_qkv"][dq + 63] = 0.0
    announce("attention backward with an infinite key")
    _, g = run_backward(dev, w, W, x, dy, idx, False)
    assert torch.isfinite(g["b_qkv"][2 * dq:]).all() and torch.isfinite(g["w_qkv"][2 * dq:]).all()
    assert not torch.isfinite(g["w_qkv"][:dq]).all()  # the key was infinite: queries' gradients hold 0 x inf
