"""Grids of bf16 projection tiles around the sizes where their form changes:
at most one workgroup per CU (64 x 64 tiles, or the four-stage ring), with
reductions long enough to be split between two to four workgroups per tile or
too short, one row past a tile and past the chip, a NeoX layer whose up
projection shares the chip with QKV, and large tiles cut in pieces. Each layer is held to the oracle
or to the unsplit grid at the bf16 tolerance. Without the split, these
forms multiply in the order of the two-stage loop, so their results are bitwise
those of one tile per workgroup; the split adds its pieces in a fixed order,
so repeated runs are equal.
"""
import pytest
import torch

import paper_2607_21291_amd as P
import synthetic as S

from gpu_util import TOL, announce, check_layer, rel_inf, run_layer, to_np, workload

pytestmark = pytest.mark.gpu


def _w(block, d, hq, hkv, hd, f, B, T):
    base = workload("neox_bf16_small" if block == S.NEOX else "qwen_bf16_small")
    return base.replace(name="grid", d_model=d, n_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=f,
                        rotary_dims=hd if block == S.QWEN else hd // 4, batch=B, seq=T)


# the last entry: whether a projection is cut in pieces
CASES = [
    (S.QWEN, 512, 8, 2, 64, 1472, 1, 140, 127, False),   # 64 x 64 tiles, down: 23 k-tiles
    (S.QWEN, 512, 8, 2, 64, 1536, 1, 140, 128, False),   # 24
    (S.QWEN, 512, 8, 2, 64, 2112, 1, 140, 129, False),   # 33, one row past a tile
    (S.QWEN, 640, 5, 1, 128, 2560, 2, 140, 129, False),  # heads of 128: QKV on the 128 x 128 ring
    (S.QWEN, 512, 8, 2, 64, 2048, 1, 1030, 1024, False),  # gate|up: 256 tiles, one per CU
    (S.QWEN, 512, 8, 2, 64, 2048, 1, 1030, 1025, False),  # 288: past it
    (S.QWEN, 1536, 12, 2, 128, 2560, 1, 800, 769, False),  # down: 64 x 64 tiles, more than one per CU
    (S.QWEN, 576, 3, 1, 32, 640, 1, 70, 65, False),      # 64 x 64 tiles: one row past a tile, half a tile of columns
    (S.QWEN, 1024, 16, 4, 64, 1024, 1, 2000, 1985, False),  # o: 497 of them, two per CU
    (S.NEOX, 512, 8, 8, 64, 2048, 1, 140, 100, False),   # up beside QKV
    (S.NEOX, 512, 8, 8, 64, 2048, 1, 1200, 1153, False),  # up and QKV: 280 tiles together
    (S.NEOX, 1536, 24, 24, 64, 2048, 1, 140, 129, False),  # reductions of 24 and 56 k-tiles
    (S.QWEN, 512, 8, 2, 64, 4032, 1, 140, 129, True),    # down: 63 k-tiles in four uneven pieces
    (S.QWEN, 640, 5, 1, 128, 3776, 2, 140, 129, True),   # 15 tiles: a padded last group of the split grid
    (S.QWEN, 1536, 12, 2, 128, 4096, 1, 800, 769, True),  # 84 tiles, which fit in two pieces but not in three
    (S.NEOX, 512, 8, 8, 64, 3712, 1, 140, 100, True),    # both operands change within the second piece
]


GATED = [(c, P.FLAG_GATE) for c in CASES if c[-1]]  # the gated epilogue on the pieces


@pytest.mark.parametrize("case,flags", [(c, 0) for c in CASES] + GATED,
                         ids=lambda c: f"{c[0]}-d{c[1]}-f{c[5]}-B{c[6]}-k{c[8]}" if isinstance(c, tuple) else str(c))
def test_grid(dev, monkeypatch, case, flags):
    *shape, k, split = case
    w = _w(*shape)
    W = S.layer_weights(w, 0)
    x = S.hidden_states(w)
    announce(f"tile grid {case} flags={flags}")
    y, scores, idx = run_layer(dev, w, W, x, k, flags=flags)
    check_layer(w, W, x, y, scores, idx, k, gate=bool(flags))
    y2, _, _ = run_layer(dev, w, W, x, k, flags=flags)
    assert torch.equal(y, y2)
    monkeypatch.setenv("DSF_GEMM_TAIL", "0")
    announce(f"unsplit {case}")
    yu, _, _ = run_layer(dev, w, W, x, k, flags=flags)
    assert torch.equal(y, yu) != split  # pieces round differently, the other forms alike
    monkeypatch.setenv("DSF_GEMM_SCHEDULE", "classic")
    yc, _, _ = run_layer(dev, w, W, x, k, flags=flags)
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


@pytest.mark.parametrize("d,f,T,k", [(512, 8192, 300, 299), (1792, 2560, 2600, 2561), (2560, 4096, 2500, 2496)])
def test_large_tiles_in_pieces(dev, monkeypatch, d, f, T, k):
    # large tiles that leave CUs idle, forced: the down projection in four
    # pieces (4 tiles), three (77) and two (100), against the unsplit grid
    w = _w(S.QWEN, d, 8, 2, 64, f, 1, T)
    W = S.layer_weights(w, 0)
    x = S.hidden_states(w)
    monkeypatch.setenv("DSF_GEMM_TILE", "large")
    announce(f"large tiles in pieces d={d} f={f} k={k}")
    y, scores, idx = run_layer(dev, w, W, x, k)
    if d == 512:
        check_layer(w, W, x, y, scores, idx, k)
    y2, _, _ = run_layer(dev, w, W, x, k)
    assert torch.equal(y, y2)
    monkeypatch.setenv("DSF_GEMM_TAIL", "0")
    yu, _, _ = run_layer(dev, w, W, x, k)
    assert rel_inf(to_np(y) - to_np(x), to_np(yu) - to_np(x)) < TOL[w.dtype]
    assert not torch.equal(y, yu)  # the split ran (it rounds differently)


def test_large_tiles_chosen_in_pieces(dev, monkeypatch):
    # 1300 Qwen2.5-1.5B rows: the rule takes large tiles in pieces for the down projection
    w = S.WORKLOADS["qwen15b"].replace(batch=1, seq=1400, n_layers=1)
    W = S.layer_weights(w, 0)
    x = S.hidden_states(w)
    announce("large tiles chosen in pieces")
    y, _, idx = run_layer(dev, w, W, x, 1300)
    monkeypatch.setenv("DSF_GEMM_TAIL", "0")
    yu, _, _ = run_layer(dev, w, W, x, 1300)
    # no grid of 128 x 128 tiles of this layer has room for two pieces per
    # tile, so only large tiles in pieces round differently without the split
    assert not torch.equal(y, yu)
    monkeypatch.delenv("DSF_GEMM_TAIL")
    monkeypatch.setenv("DSF_GEMM_TILE", "small")
    ys, _, idxs = run_layer(dev, w, W, x, 1300)
    assert torch.equal(idx, idxs)
    assert rel_inf(to_np(y) - to_np(x), to_np(ys) - to_np(x)) < TOL[w.dtype]
