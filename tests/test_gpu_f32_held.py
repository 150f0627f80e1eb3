"""fp32 passes with the weights held in registers: the rounds of 256 elements per wave and both sides of their limit (either pass), waves
without a step in the last round, tiles of rows and pairs that are not full, several tiles of pairs per workgroup and per
segment, one and two tiles of rows in the down pass, work items, and segments of one or two pairs beside larger ones."""
import pytest
import torch

from oracle import moespec_oracle as O
from paper_2602_16052_amd import binding as mb
from paper_2602_16052_amd import workloads as wl

from gpu_common import (assert_out_close, assert_routing_equal, desc_of, oracle_weights, out_to_numpy, to_device,
                        upload_weights)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,N,k,F,M,B", [(32, 2, 1, 252, 3, 2), (256, 2, 2, 28, 16, 2), (260, 2, 2, 36, 17, 2), (288, 3, 1, 20, 33, 2),
                                         (508, 2, 2, 512, 65, 2), (516, 2, 1, 544, 40, 1), (764, 2, 2, 772, 20, 2),
                                         (768, 3, 2, 768, 49, 2), (772, 2, 2, 516, 31, 2), (48, 5, 3, 260, 7, 4),
                                         (2052, 4, 2, 132, 35, 4), (140, 4, 2, 1024, 300, 3), (1040, 8, 2, 300, 270, 8),
                                         (528, 40, 2, 64, 60, 30), (32, 2, 1, 252, 18, 2), (256, 2, 2, 28, 17, 2), (48, 5, 3, 260, 19, 4),
                                         (1056, 6, 2, 36, 16, 6), (36, 40, 2, 208, 60, 40), (36, 40, 2, 208, 60, 39)])
@pytest.mark.parametrize("policy", [mb.TRUNCATE, mb.SUBSTITUTE])
def test_f32_held_weights(d, N, k, F, M, B, policy, alpha=0.8):
    print(f"case d={d} N={N} k={k} F={F} M={M} B={B} policy={policy}", flush=True)
    if policy == mb.SUBSTITUTE and B < k:
        B = k
    cfg = wl.small_config("held", "f32", d=d, n_experts=N, top_k=k, d_ff=F, M=M, bias_alpha=alpha, seed=d + M)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    h_d, W_d, ws = to_device(h), upload_weights(W), mb.alloc_workspace(desc, M)
    ref = O.layer_forward(wl.as_f32(h), oracle_weights(W), k, cfg.renorm, B, policy)
    out, taps = mb.moespec_layer_forward(desc, W_d, h_d, B, policy, ws, taps=True)
    staged = mb.moespec_expert_ffn(desc, W_d, h_d, taps["seg_expert"], taps["seg_off"], taps["perm"], taps["tok_ids"],
                                   taps["tok_w"], ws)
    torch.cuda.synchronize()
    assert_routing_equal(taps, ref, B)
    assert_out_close(out_to_numpy(out), ref["out"], "f32")
    assert torch.equal(staged, out)  # the order of the sums does not depend on the route to the pass


@pytest.mark.parametrize("d,N,k,F,M,B", [(64, 3, 2, 772, 5, 3), (20, 4, 2, 800, 70, 4), (36, 5, 3, 1020, 17, 4), (64, 3, 2, 1024, 65, 3),
                                         (64, 3, 2, 1028, 65, 3), (448, 5, 2, 964, 40, 4), (452, 5, 2, 964, 40, 4),
                                         (68, 6, 2, 900, 290, 5)])
@pytest.mark.parametrize("policy", [mb.TRUNCATE, mb.SUBSTITUTE])
def test_f32_held_weights_of_few_rows(d, N, k, F, M, B, policy):
    """The down pass of up to 112 workgroups, which holds up to 1024 elements: both sides of either limit, waves without a step in the
    fourth round, and segments that four workgroups share."""
    test_f32_held_weights(d, N, k, F, M, B, policy)


@pytest.mark.parametrize("d,N,k,F,M,B", [(48, 64, 1, 60, 80, 64), (96, 64, 2, 520, 120, 50), (48, 128, 1, 256, 200, 128), (516, 60, 1, 48, 255, 40),
                                         (36, 256, 2, 708, 363, 256), (108, 256, 1, 148, 700, 128), (64, 64, 8, 260, 200, 64)])
@pytest.mark.parametrize("alpha", [0.2, 4.0])
@pytest.mark.parametrize("policy", [mb.TRUNCATE, mb.SUBSTITUTE])
def test_f32_held_long_segments(d, N, k, F, M, B, alpha, policy):
    """Many short segments and, with alpha = 4, one of nearly all tokens (or its pieces), which up to four workgroups share."""
    test_f32_held_weights(d, N, k, F, M, B, policy, alpha)
