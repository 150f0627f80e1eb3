"""GPU parity when the router logits span hundreds to thousands: hidden rows scaled by up to 3000, so that
most routing probabilities underflow to exact zeros or denormals in the fp64 softmax (Eq. 1).  Routing must
stay bit-exact (zeros tie to the lowest id), outputs within tolerance relative to their scale, and a substitution
set of zero probability mass for a token must give NaN weights and a NaN output row on both sides."""
import numpy as np
import pytest
import torch

from oracle import moespec_oracle as O
from paper_2602_16052_amd import binding as mb
from paper_2602_16052_amd import workloads as wl

from gpu_common import TOL, assert_routing_equal, desc_of, oracle_weights, out_to_numpy, to_device, upload_weights

pytestmark = pytest.mark.gpu

CASES = [("bf16", 256, 64, 8, 128, 48, "softmax"),     # fused prologue, every workgroup rebuilds the table
         ("bf16", 128, 130, 4, 128, 200, "softmax"),   # table beyond the LDS, ragged expert count: staged kernels
         ("f32", 64, 16, 2, 32, 20, "softmax"),        # fp32 operands
         ("bf16", 256, 40, 6, 256, 130, "sigmoid"),
         ("bf16", 128, 64, 8, 128, 600, "softmax"),    # more tokens than the fused prologue takes: staged kernels
         ("bf16", 128, 70, 4, 128, 100, "softmax")]    # fused prologue, row-wise gate kernel, ragged expert count


@pytest.mark.parametrize("dtype,d,N,k,F,M,gate", CASES)
def test_underflowing_softmax_keeps_parity(dtype, d, N, k, F, M, gate):
    cfg = wl.small_config("extreme", dtype, d=d, n_experts=N, top_k=k, d_ff=F, M=M, budgets=(k, N // 2, N), seed=7,
                          gate=gate)
    scale = np.array([0.01, 1.0, 30.0, 100.0, 300.0, 1e3, 3e3], dtype=np.float32)[np.arange(M) % 7][:, None]
    h = wl.store(wl.as_f32(wl.hidden_states(cfg)) * scale, dtype)
    W = wl.layer_weights(cfg)
    desc = desc_of(cfg)
    h_d, W_d, ws = to_device(h), upload_weights(W), mb.alloc_workspace(desc, M)
    h_o, W_o = wl.as_f32(h), oracle_weights(W)
    seen_zero, seen_nan = False, False
    for B in cfg.budgets:
        for policy in (mb.TRUNCATE, mb.SUBSTITUTE):
            if policy == mb.SUBSTITUTE and B < k:
                continue
            print(f"  B={B} policy={policy}", flush=True)
            out, taps = mb.moespec_layer_forward(desc, W_d, h_d, B, policy, ws, taps=True)
            torch.cuda.synchronize()
            with np.errstate(over="ignore", invalid="ignore"):
                ref = O.layer_forward(h_o, W_o, k, cfg.renorm, B, policy, gate=gate)
            seen_zero |= bool((ref["probs"] == 0).any())
            assert_routing_equal(taps, ref, B)          # NaN weights compare equal position by position
            got, want = out_to_numpy(out), ref["out"]
            nan_rows = np.isnan(want).any(axis=1)
            assert np.array_equal(np.isnan(got).any(axis=1), nan_rows), "NaN rows differ"
            assert np.array_equal(nan_rows, np.isnan(ref["tok_w"]).any(axis=1))
            seen_nan |= bool(nan_rows.any())
            ok = ~nan_rows
            assert np.all(np.isfinite(got[ok]))
            if ok.any():
                # rows differ in scale by 3e5: each row against its own magnitude
                row_scale = np.maximum(np.max(np.abs(want[ok]), axis=1, keepdims=True), 1.0)
                assert np.max(np.abs(got[ok] - want[ok]) / row_scale) <= TOL[dtype]
    if gate == "softmax":
        assert seen_zero, "the case was meant to underflow"
    if gate == "softmax" and cfg.renorm:
        assert seen_nan, "the case was meant to reach a zero-mass substitution set"


@pytest.mark.parametrize("dtype,N,M,gate", [("bf16", 64, 7, "softmax"), ("bf16", 64, 1030, "softmax"), ("f32", 40, 33, "softmax"),
                                            ("f32", 250, 9, "softmax"), ("bf16", 257, 5, "softmax"), ("bf16", 40, 20, "sigmoid")])
def test_one_nan_logit_is_not_swallowed(dtype, N, M, gate):
    """A NaN in one expert's router bias (one in a router row: every token) makes the softmax of every token NaN, whatever
    kernel evaluates it; with the sigmoid gate it is that expert's score alone.  An expert masked with -inf gets 0."""
    print(f"case {dtype} N={N} M={M} {gate}", flush=True)
    cfg = wl.small_config("nan_bias", dtype, d=64, n_experts=N, top_k=3, d_ff=32, M=M, seed=M, gate=gate)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    W["b_router"][1] = -np.inf
    h_d, ws = to_device(h), mb.alloc_workspace(desc, M)
    W_o = oracle_weights(W)
    want, ids, _ = O.route(wl.as_f32(h), W_o["w_router"], W_o["b_router"], 3, cfg.renorm, gate)
    assert np.all(want[:, 1] == 0.0)
    masked = mb.moespec_route(desc, upload_weights(W), h_d, ws)
    torch.cuda.synchronize()
    np.testing.assert_allclose(masked["probs"].cpu().numpy(), want, rtol=1e-11, atol=1e-300)
    assert np.array_equal(masked["topk_ids"].cpu().numpy(), ids)
    bad = N // 2
    W_nan = dict(W, b_router=W["b_router"].copy())
    W_nan["b_router"][bad] = np.nan
    W_row = dict(W, w_router=W["w_router"].copy())
    W_row["w_router"][bad, 5] = 0x7FC0 if dtype == "bf16" else np.nan
    for W_bad in (W_nan, W_row):
        W_d = upload_weights(W_bad)
        r = mb.moespec_route(desc, W_d, h_d, ws)
        _, taps = mb.moespec_layer_forward(desc, W_d, h_d, N, mb.TRUNCATE, ws, taps=True)
        torch.cuda.synchronize()
        for g in (r["probs"].cpu().numpy(), taps["probs"].cpu().numpy()):
            if gate == "softmax":
                assert np.all(np.isnan(g))
            else:
                assert np.all(np.isnan(g[:, bad])) and np.all(np.isfinite(np.delete(g, bad, axis=1)))
