"""fp32 layers where their kernels can go wrong: rows that are no multiple of a wave's 8 (4 gate) rows, K below and just
above a wave's 64 elements, hidden sizes that end inside a block of the router projection, segments of 1, 4, 5, 8, 9 and
more pairs, more pair tiles than workgroups share, and a table beyond the fused prologue."""
import pytest
import torch

from oracle import moespec_oracle as O
from paper_2602_16052_amd import binding as mb
from paper_2602_16052_amd import workloads as wl

from gpu_common import (assert_out_close, assert_routing_equal, desc_of, oracle_weights, out_to_numpy, to_device,
                        upload_weights)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,N,k,F,M,B", [(4, 3, 1, 4, 1, 2), (36, 2, 2, 12, 4, 2), (60, 2, 2, 68, 5, 2),
                                         (64, 2, 2, 64, 8, 2), (68, 2, 2, 132, 9, 2), (132, 7, 3, 28, 33, 5),
                                         (100, 4, 2, 52, 300, 3), (48, 300, 5, 20, 11, 40)])
@pytest.mark.parametrize("policy", [mb.TRUNCATE, mb.SUBSTITUTE])
def test_f32_layers(d, N, k, F, M, B, policy):
    print(f"case d={d} N={N} k={k} F={F} M={M} B={B} policy={policy}", flush=True)
    cfg = wl.small_config("f32", "f32", d=d, n_experts=N, top_k=k, d_ff=F, M=M, bias_alpha=0.8, seed=d + M)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    h_d, W_d, ws = to_device(h), upload_weights(W), mb.alloc_workspace(desc, M)
    ref = O.layer_forward(wl.as_f32(h), oracle_weights(W), k, cfg.renorm, B, policy)
    out, taps = mb.moespec_layer_forward(desc, W_d, h_d, B, policy, ws, taps=True)
    staged = mb.moespec_expert_ffn(desc, W_d, h_d, taps["seg_expert"], taps["seg_off"], taps["perm"], taps["tok_ids"],
                                   taps["tok_w"], ws)
    torch.cuda.synchronize()
    assert_routing_equal(taps, ref, B)
    assert_out_close(out_to_numpy(out), ref["out"], "f32")
    assert torch.equal(staged, out)
