"""The staged layer call where its kernels change form: sums over tokens beside the gate (workgroups of 8 and of 16 tokens, the most
of either, rows that end inside a workgroup, up to 64, 128 and 256 experts, sums that don't fit beside act), pairs grouped from held ids or
loaded again, and the sum over slots (2, 4 and 8 rows at a time with remainders, in one copy and in the copies of a split
down pass)."""
import numpy as np
import pytest
import torch

from oracle import moespec_oracle as O
from paper_2602_16052_amd import binding as mb
from paper_2602_16052_amd import workloads as wl

from gpu_common import (assert_out_close, assert_routing_equal, desc_of, oracle_weights, out_to_numpy, to_device,
                        upload_weights)

pytestmark = pytest.mark.gpu


def layer(dtype, d, N, k, F, M, B, policy, gate="softmax"):
    print(f"case {dtype} d={d} N={N} k={k} F={F} M={M} B={B} policy={policy} {gate}", flush=True)
    cfg = wl.small_config("staged", dtype, d=d, n_experts=N, top_k=k, d_ff=F, M=M, bias_alpha=0.8, seed=M + N + k, gate=gate)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    h_d, W_d, ws = to_device(h), upload_weights(W), mb.alloc_workspace(desc, M)
    ref = O.layer_forward(wl.as_f32(h), oracle_weights(W), k, cfg.renorm, B, policy, gate=gate)
    out, taps = mb.moespec_layer_forward(desc, W_d, h_d, B, policy, ws, taps=True)
    plain = mb.moespec_layer_forward(desc, W_d, h_d, B, policy, ws)
    torch.cuda.synchronize()
    assert_routing_equal(taps, ref, B)
    assert_out_close(out_to_numpy(out), ref["out"], dtype, scale_aware=dtype == "bf16")
    assert torch.equal(out, plain)
    return desc, h_d, W_d, ws


@pytest.mark.parametrize("M,N,k,F,gate", [(257, 64, 2, 32, "softmax"), (263, 3, 1, 32, "sigmoid"), (1024, 65, 2, 64, "softmax"),
                                          (1025, 128, 2, 64, "sigmoid"), (1031, 64, 2, 32, "softmax"), (1024, 256, 4, 64, "softmax"),
                                          (1039, 200, 4, 64, "sigmoid"), (2048, 130, 3, 64, "softmax"), (2049, 129, 3, 64, "softmax"),
                                          (2049, 128, 2, 64, "softmax"), (4096, 17, 2, 32, "softmax"), (4097, 17, 2, 32, "softmax"),
                                          (300, 200, 1, 32, "softmax")])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_sums_beside_the_gate(M, N, k, F, gate, dtype):
    layer(dtype, 32, N, k, F, M, max(k, N // 3), mb.SUBSTITUTE, gate)


@pytest.mark.parametrize("dtype,M,N,k", [("bf16", 257, 64, 4), ("f32", 300, 200, 2), ("bf16", 2049, 17, 3)])
@pytest.mark.parametrize("policy", [mb.TRUNCATE, mb.SUBSTITUTE])
def test_shortlist_of_the_caller(dtype, M, N, k, policy):
    """Sums over tokens are only made where the scores are handed out."""
    print(f"case {dtype} N={N} k={k} M={M} policy={policy}", flush=True)
    cfg = wl.small_config("staged_ext", dtype, d=64, n_experts=N, top_k=k, d_ff=64, M=M, bias_alpha=0.8, seed=M + N)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    ext = list(range(N - 1, N // 2, -1))
    h_d, W_d, ws, ext_d = to_device(h), upload_weights(W), mb.alloc_workspace(desc, M), torch.tensor(ext, dtype=torch.int32, device="cuda")
    ref = O.layer_forward(wl.as_f32(h), oracle_weights(W), k, cfg.renorm, len(ext), policy, ext_shortlist=ext)
    plain = mb.moespec_layer_forward(desc, W_d, h_d, len(ext), policy, ws, ext_shortlist=ext_d)
    out, taps = mb.moespec_layer_forward(desc, W_d, h_d, len(ext), policy, ws, ext_shortlist=ext_d, taps=True)
    torch.cuda.synchronize()
    assert_routing_equal(taps, ref, len(ext))
    assert_out_close(out_to_numpy(out), ref["out"], dtype)
    assert torch.equal(out, plain)


@pytest.mark.parametrize("M,k", [(256, 8), (255, 7), (1, 8), (257, 7), (227, 9), (256, 9)])
@pytest.mark.parametrize("policy", [mb.TRUNCATE, mb.SUBSTITUTE])
def test_pairs_grouped(M, k, policy):
    layer("bf16", 64, 257, k, 64, M, 90, policy)  # more experts than the fused prologue takes


@pytest.mark.parametrize("dtype,F", [("bf16", 64), ("bf16", 4096), ("bf16", 8192), ("f32", 64)])  # 1, 2, 4, 1 copies
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9, 17])
@pytest.mark.parametrize("policy", [mb.TRUNCATE, mb.SUBSTITUTE])
def test_sum_over_slots(dtype, F, k, policy):
    N, M, B = k + 3, 5, k + 1
    desc, h, W, ws = layer(dtype, 96, N, k, F, M, B, policy)
    # a stack that scales the inputs of its layers writes the scaled rows from the same sum
    got = mb.moespec_stack_forward(desc, [W, W], h.clone(), B, policy, ws, pre_norm=True)
    want = h
    for _ in range(2):
        x = mb.moespec_rms_scale(desc, want)
        want = mb.moespec_layer_forward(desc, W, x, B, policy, ws, residual=want)
    torch.cuda.synchronize()
    assert torch.equal(got[0] if isinstance(got, tuple) else got, want)
