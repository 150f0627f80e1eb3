"""The fused prologue where its forms change: tables that every workgroup rebuilds from 4 x 4 tiles of the projection (remainders of
tokens and experts, hidden sizes that end inside a chunk of 128 elements and inside a lane's 8, more than four chunks per wave) and larger
ones of which the last kernel only sees ranks and sums over tokens (odd and full rows of ranks, parts of one to four tokens,
several lists per workgroup, candidates with equal probabilities, NaN)."""
import numpy as np
import pytest
import torch

from oracle import moespec_oracle as O
from paper_2602_16052_amd import binding as mb
from paper_2602_16052_amd import workloads as wl

from gpu_common import (assert_out_close, assert_routing_equal, desc_of, oracle_weights, out_to_numpy, routing_with_nan, to_device,
                        upload_weights)

pytestmark = pytest.mark.gpu

SMALL = [("bf16", 32, 1, 1, 1, 1), ("bf16", 96, 5, 2, 3, 4), ("bf16", 160, 7, 3, 5, 7), ("f32", 4, 5, 2, 6, 3),
         ("f32", 132, 9, 4, 17, 6), ("f32", 1028, 3, 1, 4, 2), ("bf16", 4256, 6, 2, 9, 5), ("f32", 4612, 4, 2, 5, 3),
         ("bf16", 64, 87, 8, 63, 40), ("bf16", 64, 21, 4, 255, 12), ("bf16", 128, 256, 6, 21, 200), ("f32", 72, 22, 3, 250, 7)]
LARGE = [("bf16", 64, 88, 8, 63, 40), ("bf16", 64, 22, 4, 255, 12), ("bf16", 32, 251, 6, 24, 130), ("bf16", 64, 234, 8, 256, 80),
         ("bf16", 64, 200, 8, 255, 200), ("bf16", 64, 256, 8, 256, 256),
         ("bf16", 128, 129, 8, 127, 64), ("f32", 72, 31, 3, 201, 11), ("bf16", 2048, 64, 8, 129, 16), ("f32", 36, 200, 2, 131, 70),
         # beyond the LDS as doubles: fused, under truncation alone (table, shortlist), staged (as two above)
         ("bf16", 64, 128, 8, 256, 128), ("f32", 36, 100, 4, 210, 30), ("f32", 36, 200, 2, 160, 75), ("bf16", 64, 140, 6, 250, 40),
         ("f32", 36, 200, 2, 160, 76), ("bf16", 64, 141, 8, 256, 46),
         # just within it: the same choice
         ("bf16", 64, 208, 8, 90, 183), ("f32", 36, 140, 3, 140, 130),
         # fp32 layers that stay fused, on either side of the limit of its tokens
         ("f32", 36, 200, 2, 128, 70), ("f32", 36, 146, 4, 127, 30), ("f32", 36, 146, 4, 129, 30)]


def run(dtype, d, N, k, M, B, gate="softmax", ext=None, spoil=None):
    print(f"case {dtype} d={d} N={N} k={k} M={M} B={B} {gate} ext={ext is not None}", flush=True)
    cfg = wl.small_config("forms", dtype, d=d, n_experts=N, top_k=k, d_ff=32, M=M, bias_alpha=0.7, seed=M + N, gate=gate)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    if spoil:
        spoil(h, W)
    h_d, W_d, ws = to_device(h), upload_weights(W), mb.alloc_workspace(desc, M)
    ext_d = None if ext is None else torch.tensor(ext, dtype=torch.int32, device="cuda")
    for policy in (mb.TRUNCATE, mb.SUBSTITUTE):
        n = B if ext is None else len(ext)
        out, taps = mb.moespec_layer_forward(desc, W_d, h_d, n, policy, ws, ext_shortlist=ext_d, taps=True)
        plain = mb.moespec_layer_forward(desc, W_d, h_d, n, policy, ws, ext_shortlist=ext_d)
        torch.cuda.synchronize()
        yield cfg, h, W, policy, out, plain, taps


@pytest.mark.parametrize("gate", ["softmax", "sigmoid"])
@pytest.mark.parametrize("dtype,d,N,k,M,B", SMALL + LARGE)
def test_table_forms(dtype, d, N, k, M, B, gate):
    assert ((dtype, d, N, k, M, B) in LARGE) == (M * N > 5500) and M <= 256  # the rule
    for cfg, h, W, policy, out, plain, taps in run(dtype, d, N, k, M, B, gate):
        ref = O.layer_forward(wl.as_f32(h), oracle_weights(W), k, cfg.renorm, B, policy, gate=gate)
        assert_routing_equal(taps, ref, B)
        assert_out_close(out_to_numpy(out), ref["out"], dtype)
        assert torch.equal(out, plain)


@pytest.mark.parametrize("dtype,d,N,k,M,B", [SMALL[4], LARGE[0], LARGE[7]])
def test_callers_shortlist(dtype, d, N, k, M, B):
    ext = [(7 * i + 3) % N for i in range(max(B, k))]
    assert len(set(ext)) == len(ext)
    for cfg, h, W, policy, out, plain, taps in run(dtype, d, N, k, M, B, ext=ext):
        ref = O.layer_forward(wl.as_f32(h), oracle_weights(W), k, cfg.renorm, len(ext), policy, ext_shortlist=ext)
        assert_routing_equal(taps, ref, len(ext))
        assert torch.equal(out, plain)


@pytest.mark.parametrize("dtype,d,N,k,M,B", [SMALL[8], LARGE[0], LARGE[6]])
def test_equal_probabilities_go_to_the_lowest_id(dtype, d, N, k, M, B):
    def twins(h, W):  # experts i and i + N / 2 alike; every second token repeats the one before
        half = N // 2
        W["w_router"][half:2 * half] = W["w_router"][:half]
        if W["b_router"] is not None:
            W["b_router"][half:2 * half] = W["b_router"][:half]
        h[1::2] = h[:2 * (M // 2):2]

    for cfg, h, W, policy, out, plain, taps in run(dtype, d, N, k, M, B, spoil=twins):
        ref = O.layer_forward(wl.as_f32(h), oracle_weights(W), k, cfg.renorm, B, policy)
        assert_routing_equal(taps, ref, B)


@pytest.mark.parametrize("gate", ["softmax", "sigmoid"])
@pytest.mark.parametrize("dtype,d,N,k,M,B", [SMALL[8], LARGE[0], LARGE[6]])
def test_a_nan_expert_claims_a_slot_and_no_pair(dtype, d, N, k, M, B, gate):
    """A router bias that is NaN: under softmax every probability is NaN, under sigmoid that of one expert.  A NaN candidate claims slot
    0 (whose weight makes the token's output NaN unless the slot is dropped), and is in no pair list; the output of a token is finite
    exactly where none of its slots is NaN."""
    bad = 5

    def nan_bias(h, W):
        W["b_router"][bad] = np.nan

    for with_bad in (True, False):
        ext = [i for i in range(B + 1) if i != bad] + ([bad] if with_bad else [])
        for cfg, h, W, policy, out, plain, taps in run(dtype, d, N, k, M, B, gate, ext=ext, spoil=nan_bias):
            ids, w = taps["tok_ids"].cpu().numpy(), taps["tok_w"].cpu().numpy()
            want_ids, want_w = routing_with_nan(taps["probs"].cpu().numpy(), k, ext, policy, cfg.renorm)
            assert np.array_equal(ids, want_ids)
            np.testing.assert_allclose(w, want_w, rtol=1e-6, atol=1e-12)  # NaN in the same places
            assert torch.equal(out.view(torch.uint8), plain.view(torch.uint8))
            off, seg = taps["seg_off"].cpu().numpy(), taps["seg_expert"].cpu().numpy()
            sizes = {int(e): int(off[i + 1] - off[i]) for i, e in enumerate(seg) if e >= 0}
            assert sizes.get(bad, 0) == 0
            rows = np.isnan(out_to_numpy(out)).any(axis=1)
            assert np.array_equal(rows, np.isnan(w).any(axis=1))
            if gate == "softmax":
                assert sum(sizes.values()) == 0 and np.all(rows)
            elif with_bad:
                assert np.all(ids[:, 0] == bad) and np.all(rows)
            elif policy == mb.SUBSTITUTE:
                assert not np.any(rows)
