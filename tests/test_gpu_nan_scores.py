"""A NaN hidden row makes every aggregate score NaN.  They rank by id then, on every path and in every workgroup alike: the
shortlist is the B lowest ids, none of its copies reaches past its end, and the tokens of finite rows come out as with that shortlist
given by the caller.  Probabilities that are NaN claim slot 0 of their token on every path alike."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import moespec_oracle as O
from paper_2602_16052_amd import binding as mb
from paper_2602_16052_amd import workloads as wl

from gpu_common import assert_out_close, desc_of, oracle_weights, out_to_numpy, routing_with_nan, to_device, upload_weights

pytestmark = pytest.mark.gpu

GUARD = 64


def guarded(n, dtype):
    return torch.full((n + GUARD,), -77, dtype=dtype, device="cuda")


# tables rebuilt by every workgroup, ranks in their place (tokens and lists in workgroups of their own, or in the same ones), staged: a
# wave per token, a workgroup per token
@pytest.mark.parametrize("dtype,d,N,k,M,B", [("bf16", 64, 128, 4, 20, 8), ("f32", 64, 256, 3, 21, 5), ("bf16", 64, 64, 8, 7, 64),
                                             ("bf16", 64, 128, 4, 60, 8), ("bf16", 64, 128, 8, 250, 16), ("f32", 32, 64, 4, 300, 6),
                                             ("bf16", 64, 128, 2, 257, 128), ("bf16", 64, 300, 4, 30, 8), ("f32", 32, 130, 4, 300, 9)])
@pytest.mark.parametrize("policy", [mb.TRUNCATE, mb.SUBSTITUTE])
def test_shortlist_of_nan_scores(dtype, d, N, k, M, B, policy):
    print(f"case {dtype} d={d} N={N} k={k} M={M} B={B} policy={policy}", flush=True)
    cfg = wl.small_config("nan_scores", dtype, d=d, n_experts=N, top_k=k, d_ff=32, M=M, bias_alpha=0.4, seed=M + N)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    bad = M // 2
    fine = np.arange(M) != bad
    S = list(range(B))
    ref = O.layer_forward(wl.as_f32(h)[fine], oracle_weights(W), k, cfg.renorm, B, policy, ext_shortlist=S)
    h_d, W_d, ws = to_device(h), upload_weights(W), mb.alloc_workspace(desc, M)
    h_d[bad, 3] = float("nan")
    ws.fill_(0xff)  # rows of pairs that nobody computes are NaN

    shapes = dict(probs=(M * N, torch.float64), scores=(N, torch.float64), budget_ids=(B, torch.int32), tok_ids=(M * k, torch.int32),
                  tok_w=(M * k, torch.float32), seg_expert=(B, torch.int32), seg_off=(B + 1, torch.int32),
                  perm=(M * k, torch.int32), n_loaded=(1, torch.int32))
    taps = {key: guarded(n, dt) for key, (n, dt) in shapes.items()}
    out = torch.empty_like(h_d)
    cd, cw = desc.c(), mb._weights(desc, W_d, True, True)
    ctaps = mb.Taps(**{key: t.data_ptr() for key, t in taps.items()})
    status = mb.load_library().moespec_layer_forward(ctypes.byref(cd), ctypes.byref(cw), h_d.data_ptr(), M, B, policy, None, None,
                                                     out.data_ptr(), ctypes.byref(ctaps), ws.data_ptr(), ws.numel(), None)
    assert status == mb.OK
    torch.cuda.synchronize()
    got = {key: t.cpu().numpy() for key, t in taps.items()}
    for key, (n, _) in shapes.items():
        assert np.all(got[key][n:] == -77), f"{key} written past its end"
    assert got["budget_ids"][:B].tolist() == S and got["seg_expert"][:B].tolist() == S
    assert np.all(np.isnan(got["scores"][:N]))
    assert np.array_equal(got["tok_ids"][:M * k].reshape(M, k)[fine], ref["tok_ids"])
    assert_out_close(out_to_numpy(out)[fine], ref["out"], dtype)

    plain = mb.moespec_layer_forward(desc, W_d, h_d, B, policy, ws)
    staged = mb.moespec_budget(desc, mb.moespec_route(desc, W_d, h_d, ws)["probs"], B, policy, ws)
    torch.cuda.synchronize()
    assert torch.equal(plain.view(torch.uint8), out.view(torch.uint8))
    assert staged["budget_ids"].tolist() == S and staged["seg_expert"].tolist() == S
    assert np.array_equal(staged["tok_ids"].cpu().numpy()[fine], ref["tok_ids"])


@pytest.mark.parametrize("N,k,M,B", [(64, 8, 10, 20), (200, 3, 9, 30), (88, 8, 63, 40), (200, 4, 100, 70), (60, 4, 300, 20), (128, 2, 300, 50),
                                     (200, 3, 600, 40), (300, 5, 20, 100), (1000, 64, 5, 200)])
@pytest.mark.parametrize("gate", ["softmax", "sigmoid"])
@pytest.mark.parametrize("renorm", [0, 1])
def test_nan_probabilities_claim_slot_0(N, k, M, B, gate, renorm):
    print(f"case N={N} k={k} M={M} B={B} {gate} renorm={renorm}", flush=True)
    cfg = wl.small_config("nan_slots", "bf16", d=32, n_experts=N, top_k=k, d_ff=64, M=M, bias_alpha=0.4, seed=M + N, gate=gate)
    h, W = wl.hidden_states(cfg), wl.layer_weights(cfg)
    desc = mb.LayerDesc(32, N, k, 64, mb.BF16, renorm, mb.GATE_SIGMOID if gate == "sigmoid" else mb.GATE_SOFTMAX)
    low, high = N // 3, N - 2  # in other blocks of 64 ids where there are several
    W["b_router"][[low, high]] = np.nan
    h_d, W_d, ws = to_device(h), upload_weights(W), mb.alloc_workspace(desc, M)
    r = mb.moespec_route(desc, W_d, h_d, ws)
    g = r["probs"].cpu().numpy()
    assert np.all(np.isnan(g[:, [low, high]]))
    want_ids, want_w = routing_with_nan(g, k, range(N), mb.TRUNCATE, renorm)
    assert np.array_equal(r["topk_ids"].cpu().numpy(), want_ids)
    np.testing.assert_allclose(r["topk_w"].cpu().numpy(), want_w, rtol=1e-6, atol=1e-12)
    others = [i for i in range(N) if i not in (low, high)]
    for ext in (others[:B], others[:B - 1] + [high], [high] + others[:B - 2] + [low], None):
        ext_d = None if ext is None else torch.tensor(ext, dtype=torch.int32, device="cuda")
        for policy in (mb.TRUNCATE, mb.SUBSTITUTE):
            b = mb.moespec_budget(desc, r["probs"], B, policy, ws, ext_shortlist=ext_d)
            out, taps = mb.moespec_layer_forward(desc, W_d, h_d, B, policy, ws, ext_shortlist=ext_d, taps=True)
            torch.cuda.synchronize()
            S = b["budget_ids"].tolist()
            assert len(set(S)) == B and taps["budget_ids"].tolist() == S
            if ext is None and gate == "softmax":
                assert S == list(range(B))
            want_ids, want_w = routing_with_nan(g, k, S, policy, renorm)
            for got in (b, taps):
                assert np.array_equal(got["tok_ids"].cpu().numpy(), want_ids)
                np.testing.assert_allclose(got["tok_w"].cpu().numpy(), want_w, rtol=1e-6, atol=1e-12)
            assert np.array_equal(np.isnan(out_to_numpy(out)).any(axis=1), np.isnan(want_w).any(axis=1))
