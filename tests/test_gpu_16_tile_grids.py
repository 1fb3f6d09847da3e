"""Grids of bf16 projection tiles around the sizes where their form changes:
at most one workgroup per CU (the four-stage ring), with reductions long
enough to be split between three or four workgroups per tile or just too
short, one row past a tile and past the chip, and a NeoX layer whose up
projection shares the chip with QKV. Each layer is held to the oracle at the
bf16 tolerance. Without the split, the ring multiplies in the order of the
two-stage loop, so its results are bitwise those of one tile per workgroup;
the split adds its pieces in a fixed order, so repeated runs are equal.
"""
import pytest
import torch

import synthetic as S

from gpu_util import announce, check_layer, run_layer, workload

pytestmark = pytest.mark.gpu


def _w(block, d, hq, hkv, hd, f, B, T):
    base = workload("neox_bf16_small" if block == S.NEOX else "qwen_bf16_small")
    return base.replace(name="grid", d_model=d, n_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=f,
                        rotary_dims=hd if block == S.QWEN else hd // 4, batch=B, seq=T)


CASES = [
    (S.QWEN, 512, 8, 2, 64, 1472, 1, 140, 127),   # down: 23 k-tiles, too few for three pieces
    (S.QWEN, 512, 8, 2, 64, 1536, 1, 140, 128),   # 24: three pieces
    (S.QWEN, 512, 8, 2, 64, 2112, 1, 140, 129),   # 33: four uneven pieces
    (S.QWEN, 640, 5, 1, 128, 2560, 2, 140, 129),  # 15 tiles: a padded last group of the split grid
    (S.QWEN, 512, 8, 2, 64, 2048, 1, 1030, 1024), # gate|up: 256 tiles, one per CU
    (S.QWEN, 512, 8, 2, 64, 2048, 1, 1030, 1025), # 288: past it
    (S.NEOX, 512, 8, 8, 64, 2048, 1, 140, 100),   # up beside QKV
    (S.NEOX, 512, 8, 8, 64, 2048, 1, 1200, 1153), # up and QKV: 280 tiles together
    (S.NEOX, 1536, 24, 24, 64, 2048, 1, 140, 129),  # reductions of 24 and 56 k-tiles
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}-d{c[1]}-f{c[5]}-B{c[6]}-k{c[8]}")
def test_grid(dev, monkeypatch, case):
    *shape, k = case
    w = _w(*shape)
    W = S.layer_weights(w, 0)
    x = S.hidden_states(w)
    announce(f"tile grid {case}")
    y, scores, idx = run_layer(dev, w, W, x, k)
    check_layer(w, W, x, y, scores, idx, k)
    y2, _, _ = run_layer(dev, w, W, x, k)
    assert torch.equal(y, y2)
    monkeypatch.setenv("DSF_GEMM_TAIL", "0")
    announce(f"unsplit {case}")
    yu, _, _ = run_layer(dev, w, W, x, k)
    monkeypatch.setenv("DSF_GEMM_SCHEDULE", "classic")
    yc, _, _ = run_layer(dev, w, W, x, k)
    assert torch.equal(yu, yc)


@pytest.mark.parametrize("B,T,k", [(1, 2100, 2049), (2, 2100, 2048), (1, 4200, 4097)])
def test_large_tile_rule(dev, B, T, k):
    # around the row counts where the 256 x 256 tiles take over (and end with
    # a split or a nearly empty round)
    w = _w(S.QWEN, 1024, 8, 2, 128, 2816, B, T)
    W = S.layer_weights(w, 0)
    x = S.hidden_states(w)
    announce(f"large tiles B={B} T={T} k={k}")
    y, scores, idx = run_layer(dev, w, W, x, k)
    check_layer(w, W, x, y, scores, idx, k, sample=[B - 1])
    y2, _, _ = run_layer(dev, w, W, x, k)
    assert torch.equal(y, y2)
