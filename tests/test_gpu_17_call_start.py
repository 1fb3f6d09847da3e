"""The launch that starts a call writes the RoPE table and clears the control
block, over sequence lengths around its workgroups. Where nothing is kept
there is no such launch: the call needs no workspace and leaves one that it
is given alone."""
import pytest
import torch

import paper_2607_21291_amd as P
import synthetic as S

from gpu_util import announce, check_layer, make_desc, run_layer, workload, workspace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k", [(1, 1), (63, 40), (65, 65), (129, 100)])
@pytest.mark.parametrize("name", ["neox_bf16_small", "tiny_neox_f32", "tiny_qwen_f32"])
def test_layer_on_a_dirty_workspace(dev, name, T, k):
    w = workload(name).replace(seq=T)
    W = S.layer_weights(w, 0)
    x = S.hidden_states(w)
    announce(f"call start {name} T={T}")
    dl = P.DeviceLayer(W, dev)
    ws = workspace(w, w.batch, T, k, dev)
    ws.fill_(0xA5)
    xd = x.to(dev)
    scores = torch.empty(w.batch, T, dtype=torch.float32, device=dev)
    idx = torch.empty(w.batch, k, dtype=torch.int32, device=dev)
    P.sparse_block_forward(make_desc(w), dl.weights, xd, k, ws, scores_out=scores, idx_out=idx)
    assert P.workspace_status(ws) == 0
    check_layer(w, W, x, xd, scores, idx, k)


def test_prefill_that_keeps_nothing(dev):
    w = workload("neox_bf16_small").replace(n_layers=2)
    dls = [P.DeviceLayer(W, dev) for W in S.stack_weights(w)]
    x = S.hidden_states(w).to(dev)
    x0 = x.clone()
    ck, cv = ([torch.zeros(w.batch, w.n_kv_heads, 8, w.head_dim, dtype=torch.bfloat16, device=dev) for _ in dls]
              for _ in range(2))
    clen = torch.full((2, w.batch), 7, dtype=torch.int32, device=dev)
    ws = torch.full((256,), 0xA5, dtype=torch.uint8, device=dev)
    announce("prefill, k = 0 in every layer")
    P.stack_prefill(make_desc(w), [dl.weights for dl in dls], [0, 0], x, ck, cv, clen, ws)
    torch.cuda.synchronize()
    assert torch.equal(x, x0) and (clen == 0).all() and (ws == 0xA5).all()


def test_current_stream_handle(dev):
    from paper_2607_21291_amd import _binding
    side = torch.cuda.Stream()
    assert _binding._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert _binding._stream(None) == side.cuda_stream
    assert _binding._stream(side) == side.cuda_stream
