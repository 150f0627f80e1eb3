"""The route stage where its dispatch changes: one slice or several of the hidden dimension (1024 / 1025 tokens),
experts around the candidates-per-lane steps and around the limit of the matrix-core projection, tokens around the limit of
the shared top-k counts, top-k of a whole wave;
and the selection counts of a batch larger than one workgroup's share."""
import numpy as np
import pytest
import torch

from oracle import moespec_oracle as O
from paper_2602_16052_amd import binding as mb
from paper_2602_16052_amd import workloads as wl

from gpu_common import desc_of, oracle_weights, to_device, upload_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,k,d,gate", [(1024, 64, 8, 64, "softmax"), (1025, 65, 8, 32, "softmax"),
                                          (1031, 17, 17, 96, "sigmoid"), (33, 128, 64, 256, "softmax"),
                                          (7, 129, 6, 512, "sigmoid"), (3, 256, 8, 1024, "softmax"),
                                          (5, 257, 8, 64, "softmax"), (2050, 1, 1, 32, "softmax"),
                                          (512, 66, 3, 32, "sigmoid"), (513, 66, 3, 32, "softmax"),
                                          (1, 253, 64, 32, "softmax"), (1025, 8, 2, 1024, "softmax"), (1100, 16, 1, 2048, "sigmoid"),
                                          # blocks per wave of the projection: 4, 5 (no loads ahead), 8 (none above 700 workgroups), 8 to 9, 12, 16
                                          (1100, 64, 4, 512, "softmax"), (1100, 64, 4, 640, "softmax"), (1100, 64, 4, 1024, "softmax"),
                                          (2900, 64, 2, 1024, "softmax"),
                                          (1100, 64, 4, 544, "softmax"), (1100, 64, 8, 1056, "softmax"), (600, 64, 4, 2080, "softmax"),
                                          (1030, 64, 2, 1184, "sigmoid"), (500, 100, 8, 4096, "softmax"), (1500, 30, 3, 3104, "softmax"),
                                          (40, 127, 127 // 2, 64, "softmax")])
def test_route_stage_edges(M, N, k, d, gate):
    check_route(M, N, k, d, gate, "bf16")


@pytest.mark.parametrize("M,N,k,d", [(1100, 64, 4, 28), (1100, 64, 8, 36), (1100, 40, 4, 132), (1100, 64, 2, 260), (1100, 64, 4, 392),
                                     (1100, 64, 6, 516), (1100, 64, 4, 548), (1100, 64, 4, 676), (1100, 64, 8, 1060),
                                     (600, 64, 4, 2084), (20, 16, 2, 4100)])
def test_route_stage_fp32_projection(M, N, k, d):
    """From none to 16 blocks of 32 elements per wave, on both sides of its sets of two blocks, in one slice and in several,
    with 0 to 28 elements behind the last block."""
    check_route(M, N, k, d, "softmax", "f32")


def check_route(M, N, k, d, gate, dtype):
    print(f"case M={M} N={N} k={k} d={d} {gate} {dtype}", flush=True)
    cfg = wl.small_config("route_edge", dtype, d=d, n_experts=N, top_k=k, d_ff=32, M=M, gate=gate, seed=M + N)
    h, W, desc = wl.hidden_states(cfg), wl.layer_weights(cfg), desc_of(cfg)
    r = mb.moespec_route(desc, upload_weights(W), to_device(h), mb.alloc_workspace(desc, M))
    counts = mb.moespec_calibration_count(desc, r["topk_ids"], torch.zeros(N, dtype=torch.int64, device="cuda"))
    torch.cuda.synchronize()
    W_o = oracle_weights(W)
    g, ids, w = O.route(wl.as_f32(h), W_o["w_router"], W_o["b_router"], k, cfg.renorm, gate)
    np.testing.assert_allclose(r["probs"].cpu().numpy(), g, rtol=1e-11, atol=1e-300)
    assert np.array_equal(r["topk_ids"].cpu().numpy(), ids)
    np.testing.assert_allclose(r["topk_w"].cpu().numpy(), w, rtol=1e-6)
    assert np.array_equal(counts.cpu().numpy(), O.calibration_counts(ids, N))


def route_us(M, N, d):
    """Time of one route stage on the GPU: replayed 20 times from a graph, so that the host's calls do not count."""
    desc = mb.LayerDesc(d, N, 2, 32, mb.BF16, True)
    W = dict(w_router=torch.randn(N, d, device="cuda").to(torch.bfloat16), b_router=torch.zeros(N, device="cuda"))
    h, ws = torch.randn(M, d, device="cuda").to(torch.bfloat16), mb.alloc_workspace(desc, M)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        mb.moespec_route(desc, W, h, ws)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(20):
            mb.moespec_route(desc, W, h, ws)
    times = []
    for _ in range(8):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        graph.replay()
        end.record()
        end.synchronize()
        times.append(start.elapsed_time(end) * 50.0)
    return min(times)


def test_the_top_k_of_many_experts_is_not_one_waves_work():
    """7 tokens x 256 experts: a single wave per token took 20.6 us against 8.4 for 64 experts, four take 11.7."""
    few, many = route_us(7, 64, 2048), route_us(7, 256, 2048)
    print(f"64 experts {few:.1f} us, 256 experts {many:.1f} us", flush=True)
    assert many < 1.9 * few


def test_few_expert_tiles_keep_their_slices_above_1024_tokens():
    """1025 tokens x 8 experts are 65 output tiles; without slices of the hidden dimension each of their waves walked a
    quarter of all 4096 elements (19.3 us against 9.2 for 1024 tokens, 11.2 with them)."""
    below, above = route_us(1024, 8, 4096), route_us(1025, 8, 4096)
    print(f"1024 tokens {below:.1f} us, 1025 tokens {above:.1f} us", flush=True)
    assert above < 1.6 * below
