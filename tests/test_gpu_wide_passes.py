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
