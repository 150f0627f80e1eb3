"""fp32 layers where their kernels can go wrong: rows that are no multiple of a wave's 8 (4 gate) rows, K below and just
above a wave's 64 elements, hidden sizes that end inside a block of the router projection, segments of 1, 4, 5, 8, 9 and
more pairs, more pair tiles than workgroups share, and trees on both sides of the fused prologue's limits (experts and
tokens), with segments of several work items."""
import numpy as np
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
                                         (100, 4, 2, 52, 300, 3), (48, 300, 5, 20, 11, 40),
                                         (64, 4, 2, 32, 256, 3), (64, 4, 2, 32, 257, 3),
                                         (68, 9, 3, 44, 700, 7),
                                         # tiles of 16 rows and pairs: a K shorter than a step, remainders of rows, pairs and K
                                         (12, 3, 1, 20, 17, 3), (516, 2, 2, 24, 33, 2), (260, 1, 1, 48, 16, 1),
                                         # long rows of either pass; the largest weights of the vector form, and past them
                                         (36, 2, 2, 4100, 40, 2), (4100, 3, 2, 36, 300, 2), (1028, 2, 1, 2052, 8, 2),
                                         (1028, 2, 1, 2052, 9, 2), (1028, 2, 2, 2040, 3, 2),
                                         (300, 5, 3, 332, 1, 4), (260, 3, 3, 516, 2, 3), (256, 2, 2, 256, 3, 2),
                                         # one and two tokens among more experts than the fused prologue takes
                                         (36, 300, 3, 44, 1, 280), (68, 260, 2, 36, 2, 260)])
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


@pytest.mark.parametrize("d,N,k,F,M,B", [(36, 2, 2, 4100, 40, 2), (36, 4, 2, 2052, 300, 4), (132, 3, 1, 3076, 290, 3)])
def test_f32_two_pair_tiles(d, N, k, F, M, B):
    """Two tiles of 16 pairs per workgroup, with the fused prologue and with the staged one: segments above 128 pairs, tiles and
    pieces that end after one tile and after two."""
    assert M * k // B > 16 and -(-F // 16) * B * -(-(M * k // B) // 32) >= 512  # the rule
    for policy in (mb.TRUNCATE, mb.SUBSTITUTE):
        test_f32_layers(d, N, k, F, M, B, policy)


@pytest.mark.parametrize("d,N,k,F,M,B", [(36, 200, 2, 2052, 20, 200), (160, 128, 1, 1028, 60, 128), (36, 300, 2, 1380, 20, 300)])
def test_f32_short_rows_by_the_ten_thousand(d, N, k, F, M, B):
    """Gate/up rows of up to 160 elements and more than 24576 workgroups with few pairs: the vector form in that pass alone, with
    the prologue's lists and with work items."""
    assert M * k // B <= 6 and -(-F // 16) * B * min(-(-M // 16), 4) >= 24576  # the rule
    test_f32_layers(d, N, k, F, M, B, mb.SUBSTITUTE)


def test_f32_short_rows_count_the_segments():
    """Just below that limit by the segments, above it by the room for work items, which only the layer call has: the stage calls
    add in the same order."""
    d, N, k, F, M, B = 36, 128, 2, 752, 300, 128
    tiles, room = -(-F // 16), B + M * k // 128
    assert M * k // B <= 6 and tiles * B * 4 < 24576 <= tiles * room * 4
    test_f32_layers(d, N, k, F, M, B, mb.SUBSTITUTE)


def segment_layer(d, F, sizes, k, seed):
    """Hand-made segment tables: expert i serves sizes[i] pairs, dealt to the tokens in turn; some slots stay empty."""
    N, M = len(sizes), -(-(sum(sizes) + 3) // k)
    assert max(sizes) <= M
    cfg = wl.small_config("f32_sizes", "f32", d=d, n_experts=N, top_k=k, d_ff=F, M=M, seed=seed)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    ids = np.full(M * k, -1, dtype=np.int32)
    ids[(np.arange(sum(sizes)) % M) * k + np.arange(sum(sizes)) // M] = np.repeat(np.arange(N), sizes)
    tok_ids = ids.reshape(M, k)
    tok_w = np.where(tok_ids >= 0, np.random.default_rng(seed).uniform(0.1, 1.0, (M, k)), 0.0).astype(np.float32)
    perm = np.full(M * k, -1, dtype=np.int32)
    perm[: sum(sizes)] = np.concatenate([np.flatnonzero(ids == i) for i in range(N)])
    seg_off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    out = mb.moespec_expert_ffn(desc, upload_weights(W), to_device(h), dev(np.arange(N, dtype=np.int32)), dev(seg_off), dev(perm),
                                dev(tok_ids), dev(tok_w), mb.alloc_workspace(desc, M))
    torch.cuda.synchronize()
    W_o = oracle_weights(W)
    want = O.combine(wl.as_f32(h), tok_ids, tok_w, W_o["w_gate"], W_o["w_up"], W_o["w_down"])
    assert_out_close(out_to_numpy(out), want, "f32")


@pytest.mark.parametrize("d,F", [(4, 12), (60, 64), (64, 36), (68, 132), (508, 516), (512, 28), (516, 1024), (1028, 508)])
def test_segments_of_one_and_two_pairs(d, F):
    """They take a form of their own beside the matrix tiles: rows and K on both sides of its steps of 64 and rounds of 512 elements."""
    print(f"case d={d} F={F}", flush=True)
    segment_layer(d, F, [1, 2, 3, 2, 1, 16, 17, 2, 33], 2, d + F)


@pytest.mark.parametrize("N,B,M", [(2, 2, 16130), (300, 300, 9), (300, 260, 40)])
def test_short_segments_and_last_pieces_among_work_items(N, B, M):
    """Behind the staged prologue: 16130 tokens make 127 pieces of an expert, the last of 2 pairs, which is summed like the
    others; 300 experts serve a pair or two each."""
    print(f"case N={N} B={B} M={M}", flush=True)
    cfg = wl.small_config("f32_items", "f32", d=68, n_experts=N, top_k=2, d_ff=36, M=M, bias_alpha=0.1, seed=M)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    h_d, W_d, ws = to_device(h), upload_weights(W), mb.alloc_workspace(desc, M)
    ref = O.layer_forward(wl.as_f32(h), oracle_weights(W), 2, cfg.renorm, B, mb.SUBSTITUTE)
    out, taps = mb.moespec_layer_forward(desc, W_d, h_d, B, mb.SUBSTITUTE, ws, taps=True)
    staged = mb.moespec_expert_ffn(desc, W_d, h_d, taps["seg_expert"], taps["seg_off"], taps["perm"], taps["tok_ids"],
                                   taps["tok_w"], ws)
    torch.cuda.synchronize()
    assert_routing_equal(taps, ref, B)
    sizes = np.diff(ref["seg_off"])
    assert np.any(sizes % 127 == 1 if N == 2 else (sizes > 0) & (sizes <= 2))
    assert_out_close(out_to_numpy(out), ref["out"], "f32")
    assert torch.equal(staged, out)


def test_large_weights_and_many_experts():
    """Five tokens, more experts than the fused prologue takes, weights of 2^21 elements: the vector form of both passes on work
    items, against 64 bits and against the same form on segment arrays.  (6.5 GB of weights, made on the GPU.)"""
    d, F, N, k, M = 1448, 1452, 257, 2, 5
    assert 2 < M <= 8 and d * F >= 2 ** 21 and N > 256
    gen = torch.Generator(device="cuda").manual_seed(0)

    def normal(*shape, sigma=0.02):
        return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0.0, sigma, generator=gen)

    W = dict(w_router=normal(N, d), b_router=torch.zeros(N, device="cuda"), w_gate=normal(N, F, d), w_up=normal(N, F, d),
             w_down=normal(N, d, F))
    desc, h = mb.LayerDesc(d, N, k, F, mb.F32, True), normal(M, d, sigma=1.0)
    h[1], h[3] = h[0], h[0]  # a segment of three pairs
    ws = mb.alloc_workspace(desc, M)
    out, taps = mb.moespec_layer_forward(desc, W, h, N, mb.SUBSTITUTE, ws, taps=True)
    staged = mb.moespec_expert_ffn(desc, W, h, taps["seg_expert"], taps["seg_off"], taps["perm"], taps["tok_ids"],
                                   taps["tok_w"], ws)
    torch.cuda.synchronize()
    want = torch.zeros(M, d, dtype=torch.float64, device="cuda")
    for t in range(M):
        for s in range(k):
            e, x = int(taps["tok_ids"][t, s]), h[t].double()
            act = torch.nn.functional.silu(W["w_gate"][e].double() @ x) * (W["w_up"][e].double() @ x)
            want[t] += taps["tok_w"][t, s].double() * (W["w_down"][e].double() @ act)
    assert_out_close(out_to_numpy(out), want.cpu().numpy(), "f32")
    assert torch.equal(staged, out)


def test_one_pair_per_expert_is_a_stream_of_weights():
    """64 experts with one pair each: sixteen tokens read what two read (304 against 264 us when the pairs of sixteen took a
    tile of 16 on the matrix cores)."""
    d, F, N = 1400, 1400, 64
    gen = torch.Generator(device="cuda").manual_seed(0)

    def normal(*shape):
        return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0.0, 0.02, generator=gen)

    def ints(n):
        return torch.arange(n, dtype=torch.int32, device="cuda")

    W = dict(w_gate=normal(N, F, d), w_up=normal(N, F, d), w_down=normal(N, d, F))

    def best_us(M):
        k = N // M
        desc, h = mb.LayerDesc(d, N, k, F, mb.F32, True), normal(M, d)
        ws, tok_w, out, times = mb.alloc_workspace(desc, M), torch.ones(M, k, device="cuda"), torch.empty_like(h), []
        for _ in range(8):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(8):
                mb.moespec_expert_ffn(desc, W, h, ints(N), ints(N + 1), ints(N), ints(N).view(M, k), tok_w, ws, out=out)
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end) * 125.0)
        return min(times)

    two, sixteen = best_us(2), best_us(16)
    print(f"two tokens {two:.0f} us, sixteen {sixteen:.0f} us", flush=True)
    assert sixteen < 1.06 * two


def test_one_token_is_a_stream_of_weights():
    """One token and seven read the same two experts; the products with pairs that are not there made up the difference
    (333 against 346 us)."""
    d, F = 4096, 14336
    desc = mb.LayerDesc(d, 2, 2, F, mb.F32, True)
    gen = torch.Generator(device="cuda").manual_seed(0)

    def normal(*shape, sigma):
        return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0.0, sigma, generator=gen)

    W = dict(w_router=normal(2, d, sigma=0.02), b_router=torch.zeros(2, device="cuda"), w_gate=normal(2, F, d, sigma=0.02),
             w_up=normal(2, F, d, sigma=0.02), w_down=normal(2, d, F, sigma=0.02))

    def best_us(M):
        h, ws = normal(M, d, sigma=1.0), mb.alloc_workspace(desc, M)
        call = mb.LayerForwardCall(desc, W, h, 2, mb.SUBSTITUTE, ws, torch.empty_like(h))
        times = []
        for _ in range(8):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(8):
                call()
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end) * 125.0)
        return min(times)

    one, seven = best_us(1), best_us(7)
    print(f"one token {one:.0f} us, seven {seven:.0f} us", flush=True)
    assert one < 0.91 * seven


def test_a_large_tree_costs_no_rounds_of_its_whole_table():
    """With a workgroup per token that loads the whole table, 1024 tokens over 4 small experts were four rounds of 1024
    rows each (78 us against 20 for 256 tokens, on a shortlist of one expert with few pairs; 21 row by row)."""
    d, N, F = 64, 4, 64
    desc = mb.LayerDesc(d, N, 1, F, mb.F32, True)
    cfg = wl.small_config("table", "f32", d=d, n_experts=N, top_k=1, d_ff=F, M=1024, bias_alpha=0.0)
    W, ext = upload_weights(wl.layer_weights(cfg)), torch.zeros(1, dtype=torch.int32, device="cuda")
    W["b_router"][0] = -3.0

    def best_us(M):
        h, ws = to_device(wl.hidden_states(cfg))[:M].contiguous(), mb.alloc_workspace(desc, M)
        call = mb.LayerForwardCall(desc, W, h, 1, mb.TRUNCATE, ws, torch.empty_like(h), ext_shortlist=ext)
        times = []
        for _ in range(8):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(20):
                call()
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end) * 50.0)
        return min(times)

    small, large = best_us(256), best_us(1024)
    print(f"256 tokens {small:.0f} us, 1024 tokens {large:.0f} us", flush=True)
    assert large < 1.8 * small
