"""The grouped form of the expert passes (trees whose experts serve many pairs) at the sizes where it can go wrong:
rows that end inside a tile, K of one stage, K that ends with half a stage, pieces of exactly 96 / 97 / 128 pairs, segments
from a few pairs to several pieces; the smallest tree that takes it and the largest that does not."""
import pytest
import torch

from oracle import moespec_oracle as O
from paper_2602_16052_amd import binding as mb
from paper_2602_16052_amd import workloads as wl

from gpu_common import (assert_out_close, assert_routing_equal, desc_of, oracle_weights, out_to_numpy, to_device,
                        upload_weights)

pytestmark = pytest.mark.gpu

#        d    N   k   F   M    B  alpha
CASES = [(64, 2, 2, 64, 384, 2, 0.2),      # one stage; three pieces of 128
         (96, 5, 2, 160, 288, 4, 0.2),     # half a last stage in both passes, rows inside a tile
         (192, 2, 2, 96, 291, 2, 0.2),     # pieces of 97
         (128, 2, 2, 64, 129, 2, 0.2),     # two uneven pieces, smallest tree
         (128, 2, 2, 64, 128, 2, 0.2),     # streaming form
         (320, 12, 3, 416, 400, 12, 1.6),  # segments of every size
         (256, 40, 4, 256, 520, 33, 1.2),  # more than one round of items per XCD
         (32, 4, 2, 32, 300, 4, 0.2)]      # too narrow: streaming form


@pytest.mark.parametrize("d,N,k,F,M,B,alpha", CASES)
def test_wide_passes(d, N, k, F, M, B, alpha):
    print(f"case d={d} N={N} k={k} F={F} M={M} B={B}", flush=True)
    cfg = wl.small_config("wide", "bf16", d=d, n_experts=N, top_k=k, d_ff=F, M=M, bias_alpha=alpha, seed=M)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    h_d, W_d, ws = to_device(h), upload_weights(W), mb.alloc_workspace(desc, M)
    ref = O.layer_forward(wl.as_f32(h), oracle_weights(W), k, cfg.renorm, B, mb.SUBSTITUTE)
    out, taps = mb.moespec_layer_forward(desc, W_d, h_d, B, mb.SUBSTITUTE, ws, taps=True)
    torch.cuda.synchronize()
    assert_routing_equal(taps, ref, B)
    assert_out_close(out_to_numpy(out), ref["out"], "bf16")
    staged = mb.moespec_expert_ffn(desc, W_d, h_d, taps["seg_expert"], taps["seg_off"], taps["perm"], taps["tok_ids"],
                                   taps["tok_w"], ws)
    again = mb.moespec_layer_forward(desc, W_d, h_d, B, mb.SUBSTITUTE, ws)
    torch.cuda.synchronize()
    assert torch.equal(staged, out) and torch.equal(again, out)


@pytest.mark.parametrize("dtype,d,F,M,B", [("bf16", 128, 192, 300, 4), ("bf16", 128, 128, 600, 16), ("f32", 68, 36, 40, 6)])
def test_staged_and_wide_layers_replay_from_a_graph(dtype, d, F, M, B):
    """Captured once and replayed on other inputs with eager calls in between: every replay equals the eager result."""
    print(f"case {dtype} d={d} F={F} M={M} B={B}", flush=True)
    cfg = wl.small_config("graph", dtype, d=d, n_experts=16, top_k=4, d_ff=F, M=M, bias_alpha=0.8)
    desc, W_d = desc_of(cfg), upload_weights(wl.layer_weights(cfg))
    ws = mb.alloc_workspace(desc, M)
    inputs = [to_device(wl.hidden_states(cfg, seed=s)) for s in (0, 1, 2)]
    eager = [mb.moespec_layer_forward(desc, W_d, h, B, mb.SUBSTITUTE, ws).clone() for h in inputs]
    h_static, out_static = inputs[0].clone(), torch.empty_like(eager[0])
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        mb.LayerForwardCall(desc, W_d, h_static, B, mb.SUBSTITUTE, ws, out_static, stream=side)()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mb.LayerForwardCall(desc, W_d, h_static, B, mb.SUBSTITUTE, ws, out_static)()
    for rep in range(3):
        for h, want in zip(inputs, eager):
            h_static.copy_(h)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out_static, want), f"replay {rep} differs from the eager call"
            assert torch.equal(mb.moespec_layer_forward(desc, W_d, h, B, mb.SUBSTITUTE, ws), want)
