"""Expert passes with so few workgroups that the waves of a workgroup share K instead of the rows: K of exactly four chunks,
chunks that do not divide by four, a tail in the last wave's part, one to eight token tiles, either pass alone in that
form; and the shapes just beyond the rule."""
import numpy as np
import pytest
import torch

from oracle import moespec_oracle as O
from paper_2602_16052_amd import binding as mb
from paper_2602_16052_amd import workloads as wl

from gpu_common import (assert_out_close, assert_routing_equal, desc_of, oracle_weights, out_to_numpy, to_device,
                        upload_weights)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,N,k,F,M,B", [(512, 2, 2, 512, 16, 2), (640, 2, 2, 800, 17, 2), (1056, 3, 1, 544, 33, 3),
                                         (512, 2, 2, 64, 128, 2), (64, 2, 2, 1440, 100, 2), (544, 4, 2, 2048, 32, 4),
                                         (544, 4, 2, 2048, 33, 4), (2080, 20, 3, 96, 1, 20)])
def test_cut_walks(d, N, k, F, M, B):
    print(f"case d={d} N={N} k={k} F={F} M={M} B={B}", flush=True)
    cfg = wl.small_config("cut", "bf16", d=d, n_experts=N, top_k=k, d_ff=F, M=M, bias_alpha=0.4, seed=d + F + M)
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


def segment_layer(d, F, sizes, M, seed):
    """Hand-made segment tables: expert i serves sizes[i] tokens (top-1), rows scattered over the tree."""
    N = len(sizes)
    assert sum(sizes) <= M
    cfg = wl.small_config("cut_sizes", "bf16", d=d, n_experts=N, top_k=1, d_ff=F, M=M, seed=seed)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    rng = np.random.default_rng(seed)
    tok_ids = np.full((M, 1), -1, dtype=np.int32)
    tok_ids[rng.permutation(M)[: sum(sizes)], 0] = np.repeat(np.arange(N), sizes)
    tok_w = np.where(tok_ids >= 0, rng.uniform(0.1, 1.0, (M, 1)), 0.0).astype(np.float32)
    pairs = [np.flatnonzero(tok_ids.ravel() == i) for i in range(N)]
    perm = np.full(M, -1, dtype=np.int32)
    perm[: sum(sizes)] = np.concatenate(pairs)
    seg_off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    out = mb.moespec_expert_ffn(desc, upload_weights(W), to_device(h), dev(np.arange(N, dtype=np.int32)), dev(seg_off), dev(perm),
                                dev(tok_ids), dev(tok_w), mb.alloc_workspace(desc, M))
    torch.cuda.synchronize()
    W_o = oracle_weights(W)
    want = O.combine(wl.as_f32(h), tok_ids, tok_w, W_o["w_gate"], W_o["w_up"], W_o["w_down"])
    assert_out_close(out_to_numpy(out), want, "bf16")


@pytest.mark.parametrize("d,F", [(512, 512), (640, 544), (1184, 96), (96, 800)])
def test_pieces_on_both_sides_of_every_step(d, F):
    """Pairs where the number of token tiles that a cut walk keeps changes (one group of two tiles, two, four), and segments that
    are cut into pieces.  Empty segments behind them keep the tree out of the grouped form."""
    print(f"case d={d} F={F}", flush=True)
    sizes, M = [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 191] + [0] * 25, 1100
    assert M < 32 * len(sizes)  # fewer pairs per segment than the grouped form asks for
    pieces = sum(-(-c // 128) for c in sizes)
    cut = [K >= 512 and pieces * -(-rows // 4) <= 176 for K, rows in ((d, F // 16), (F, d // 32))]  # gate/up, down pass
    assert cut == [d >= 512, F >= 512]
    segment_layer(d, F, sizes, M, d + F)


@pytest.mark.parametrize("n,size", [(131, 2), (132, 2), (133, 2), (175, 65), (176, 65), (177, 65), (133, 64)])
def test_units_on_both_sides_of_the_limits(n, size):
    """n segments of one row tile each, the largest of `size` pairs (one of them, the rest have two): the last number of units
    whose walks are cut and the first that are not, with up to 64 pairs and with more."""
    print(f"case n={n} size={size}", flush=True)
    segment_layer(512, 32, [2] * (n - 1) + [size], 2 * n + size, n + size)


# ... and the largest tree whose tokens and pair lists have workgroups of their own, and the next
@pytest.mark.parametrize("M,B", [(1, 64), (7, 16), (15, 16), (16, 16), (200, 56), (200, 57)])
@pytest.mark.parametrize("policy", [mb.TRUNCATE, mb.SUBSTITUTE])
def test_fewer_tokens_than_shortlist_ranks(M, B, policy):
    """The fused prologue then has workgroups without a token, which only build pair lists."""
    print(f"case M={M} B={B} policy={policy}", flush=True)
    cfg = wl.small_config("ranks", "bf16", d=128, n_experts=64, top_k=8, d_ff=128, M=M, bias_alpha=0.6, seed=M)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    out, taps = mb.moespec_layer_forward(desc, upload_weights(W), to_device(h), B, policy, mb.alloc_workspace(desc, M),
                                         taps=True)
    torch.cuda.synchronize()
    ref = O.layer_forward(wl.as_f32(h), oracle_weights(W), 8, cfg.renorm, B, policy)
    assert_routing_equal(taps, ref, B)
    assert_out_close(out_to_numpy(out), ref["out"], "bf16")
