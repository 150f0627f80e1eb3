"""bf16 layers whose hidden size or expert width is no multiple of the 128-element chunk of the expert passes: one chunk
that is not full, a tail of 32, 64 and 96 elements in either pass, the K split of the down pass with a tail in its last
part, and segments for every count of token tiles; fused call, stage call and oracle."""
import pytest
import torch

from oracle import moespec_oracle as O
from paper_2602_16052_amd import binding as mb
from paper_2602_16052_amd import workloads as wl

from gpu_common import (assert_out_close, assert_routing_equal, desc_of, oracle_weights, out_to_numpy, to_device,
                        upload_weights)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,N,k,F,M,B", [(32, 3, 2, 32, 9, 2), (64, 2, 2, 96, 16, 2), (160, 2, 2, 128, 17, 2),
                                         (128, 2, 2, 192, 33, 2), (224, 2, 2, 352, 64, 2), (416, 2, 2, 288, 65, 2),
                                         (192, 9, 3, 160, 127, 5), (128, 4, 2, 4128, 20, 3), (96, 2, 1, 8288, 128, 2),
                                         (2080, 6, 2, 1056, 40, 4)])
def test_k_tails(d, N, k, F, M, B):
    print(f"case d={d} N={N} k={k} F={F} M={M} B={B}", flush=True)
    cfg = wl.small_config("tails", "bf16", d=d, n_experts=N, top_k=k, d_ff=F, M=M, bias_alpha=0.4, seed=d + F)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    h_d, W_d, ws = to_device(h), upload_weights(W), mb.alloc_workspace(desc, M)
    ref = O.layer_forward(wl.as_f32(h), oracle_weights(W), k, cfg.renorm, B, mb.SUBSTITUTE)
    out, taps = mb.moespec_layer_forward(desc, W_d, h_d, B, mb.SUBSTITUTE, ws, taps=True)
    staged = mb.moespec_expert_ffn(desc, W_d, h_d, taps["seg_expert"], taps["seg_off"], taps["perm"], taps["tok_ids"],
                                   taps["tok_w"], ws)
    torch.cuda.synchronize()
    assert_routing_equal(taps, ref, B)
    assert_out_close(out_to_numpy(out), ref["out"], "bf16")
    assert torch.equal(staged, out)


def test_infinities_beyond_the_row_end_stay_out():
    """The bytes after a row belong to the next row: infinite weights there must not reach this row's sums."""
    cfg = wl.small_config("tail_inf", "bf16", d=96, n_experts=2, top_k=1, d_ff=160, M=12, bias_alpha=0.0, seed=5)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    W["b_router"][:] = [50.0, 0.0]                       # every token goes to expert 0
    for key in ("w_gate", "w_up", "w_down"):
        W[key][1] = 0x7F80                               # +inf: the rows after expert 0's last
    ref = O.layer_forward(wl.as_f32(h), oracle_weights(W), 1, cfg.renorm, 1, mb.SUBSTITUTE)
    out = mb.moespec_layer_forward(desc, upload_weights(W), to_device(h), 1, mb.SUBSTITUTE, mb.alloc_workspace(desc, 12))
    torch.cuda.synchronize()
    assert_out_close(out_to_numpy(out), ref["out"], "bf16")
