"""The grouped form of the expert passes (trees whose experts serve many pairs) at the sizes where it can go wrong:
rows that end inside a tile, K of one stage, K that ends with half a stage, pieces on both sides of every step of its token
tiles (32, 64, 96, 128 pairs), segments from a few pairs to several pieces; the smallest tree that takes it and the largest
that does not; either pass alone in it."""
import numpy as np
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
         (192, 2, 2, 96, 288, 2, 0.2),     # pieces of 96
         (192, 2, 2, 96, 291, 2, 0.2),     # pieces of 97
         (128, 2, 2, 64, 129, 2, 0.2),     # two uneven pieces, too few units for a tree of this size: streaming form
         (1024, 2, 2, 1024, 129, 2, 0.2),  # the same with enough units, smallest tree
         (128, 2, 2, 64, 128, 2, 0.2),     # streaming form
         (64, 2, 2, 4096, 300, 2, 0.2),    # gate/up grouped, down streaming with its K cut in two
         (96, 2, 2, 8288, 260, 2, 0.2),    # ... in four, with a tail
         (2048, 2, 2, 4096, 768, 2, 0.2),  # both grouped: enough units for the long rows
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


@pytest.mark.parametrize("d,F", [(64, 160), (224, 64), (96, 96)])
def test_pieces_on_both_sides_of_every_step(d, F):
    """Hand-made segment tables for a tree that takes the grouped form: the sizes where a wave's number of token tiles
    changes, a piece of one pair, and segments that are cut into pieces of those sizes."""
    M, N, k = 450, 12, 3
    slots = [[1, 32, 33, 64, 65, 95, 160], [96, 97, 127, 130], [128]]  # pairs per expert, expert after expert, of each slot
    sizes = [n for slot in slots for n in slot]
    assert len(sizes) == N and all(sum(s) <= M for s in slots)
    cut = [-(-n // -(-n // 128)) for n in sizes]  # the longest piece of each segment
    assert {1, 32, 33, 64, 65, 80, 95, 96, 97, 127, 128} == set(cut) and sum(sizes) <= M * k and M * k >= 32 * N and M > 256
    cfg = wl.small_config("pieces", "bf16", d=d, n_experts=N, top_k=k, d_ff=F, M=M, seed=d + F)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    tok_ids, e = np.full((M, k), -1, dtype=np.int32), 0
    for s, slot in enumerate(slots):
        t0 = 7 * s
        for n in slot:
            tok_ids[np.arange(t0, t0 + n) % M, s] = e
            t0, e = t0 + n, e + 1
    tok_w = np.where(tok_ids >= 0, np.random.default_rng(d).uniform(0.1, 1.0, (M, k)), 0.0).astype(np.float32)
    pairs = [np.flatnonzero(tok_ids.ravel() == i) for i in range(N)]
    assert [p.size for p in pairs] == sizes
    perm = np.full(M * k, -1, dtype=np.int32)
    perm[: sum(sizes)] = np.concatenate(pairs)
    seg_off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    out = mb.moespec_expert_ffn(desc, upload_weights(W), to_device(h), dev(np.arange(N, dtype=np.int32)), dev(seg_off), dev(perm),
                                dev(tok_ids), dev(tok_w), mb.alloc_workspace(desc, M))
    torch.cuda.synchronize()
    W_o = oracle_weights(W)
    want = O.combine(wl.as_f32(h), tok_ids, tok_w, W_o["w_gate"], W_o["w_up"], W_o["w_down"])
    assert_out_close(out_to_numpy(out), want, "bf16")


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


@pytest.mark.parametrize("M,B", [(160, 2), (255, 4)])
def test_few_large_experts_keep_their_pace_above_128_tokens(M, B):
    """2 or 4 of 8 experts of 4096 x 14336: a down pass without a split of its long rows took 316 us for what 128 tokens
    take 147 us; the passes read the same experts, twice where a segment exceeds 128 pairs."""
    d, N, k, F = 4096, 8, 2, 14336
    desc = mb.LayerDesc(d, N, k, F, mb.BF16, True)
    gen = torch.Generator(device="cuda").manual_seed(0)

    def normal(*shape, sigma):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, sigma, generator=gen)

    W = dict(w_router=normal(N, d, sigma=0.02), b_router=torch.zeros(N, device="cuda"), w_gate=normal(N, F, d, sigma=0.02),
             w_up=normal(N, F, d, sigma=0.02), w_down=normal(N, d, F, sigma=0.02))

    def best_us(m):
        h, ws = normal(m, d, sigma=1.0), mb.alloc_workspace(desc, m)
        call = mb.LayerForwardCall(desc, W, h, B, mb.TRUNCATE, ws, torch.empty_like(h))
        times = []
        for _ in range(6):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(10):
                call()
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end) * 100.0)
        return min(times)

    base, large = best_us(128), best_us(M)
    print(f"B={B}: 128 tokens {base:.0f} us, {M} tokens {large:.0f} us", flush=True)
    assert large < 1.35 * base
