"""The budget stage at the sizes where its dispatch and its blocks change: tokens around the limit of the direct score
sum and of a score block, experts around the candidates-per-lane steps, top-k of 1 and of a whole wave, more tokens
than waves, ragged everything.  The probabilities are multiples of 2^-12, so that every sum is exact in any order and
ties are frequent: scores, shortlist, routing and segments must equal the oracle's exactly."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import moespec_oracle as O
from paper_2602_16052_amd import binding as mb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,k,B", [(1, 1, 1, 1), (1, 64, 8, 9), (128, 64, 8, 33), (129, 65, 1, 2), (127, 128, 8, 64),
                                     (130, 129, 6, 77), (257, 257, 5, 200), (1025, 5, 3, 4), (2100, 64, 8, 64),
                                     (40, 1024, 64, 700), (300, 3, 3, 3), (1, 257, 1, 1), (129, 513, 8, 300), (600, 320, 9, 60), (512, 129, 4, 40), (256, 64, 8, 20), (257, 128, 2, 30), (256, 128, 8, 90), (513, 129, 4, 40),
                                     (63, 256, 8, 64),                                      (1040, 1024, 64, 700)])
@pytest.mark.parametrize("policy", [mb.TRUNCATE, mb.SUBSTITUTE])
def test_budget_stage_edges(M, N, k, B, policy):
    print(f"case M={M} N={N} k={k} B={B} policy={policy}", flush=True)
    r = np.random.default_rng(M * 7 + N)
    g = r.integers(0, 1 << 12, size=(M, N)).astype(np.float64) / (1 << 12)
    g[:, : N // 2] *= r.integers(0, 2, size=(M, N // 2))  # exact zeros: experts that underflow
    desc = mb.LayerDesc(32, N, k, 32, mb.BF16, True)
    ws = mb.alloc_workspace(desc, M)
    b = mb.moespec_budget(desc, torch.from_numpy(g).cuda(), B, policy, ws)
    torch.cuda.synchronize()
    ids = np.array([O.top_k(row, k) for row in g], dtype=np.int32)
    w = np.array([O.mixing_weights(row, i, True) for row, i in zip(g, ids)])
    ref = O.budget(g, ids, w, B, policy, k, True)
    got = {key: val.cpu().numpy() for key, val in b.items()}
    assert np.array_equal(got["scores"], ref["scores"])
    assert np.array_equal(got["budget_ids"], ref["S"])
    assert np.array_equal(got["tok_ids"], ref["tok_ids"])
    assert np.array_equal(got["seg_expert"], ref["seg_expert"])
    assert np.array_equal(got["seg_off"], ref["seg_off"])
    P = int(ref["seg_off"][-1])
    assert np.array_equal(got["perm"][:P], ref["perm"]) and np.all(got["perm"][P:] == -1)
    assert int(got["n_loaded"][0]) == int(np.count_nonzero(np.diff(ref["seg_off"])))
    # fp32 storage of an fp64 quotient: half an ulp
    np.testing.assert_allclose(got["tok_w"], ref["tok_w"], rtol=2.0 ** -24, atol=0)


@pytest.mark.parametrize("M,N,k,B", [(5, 6, 2, 3), (63, 64, 8, 20), (130, 65, 3, 7), (40, 130, 6, 40), (300, 257, 5, 90),
                                     (9, 1000, 17, 130)])
@pytest.mark.parametrize("policy", [mb.TRUNCATE, mb.SUBSTITUTE])
def test_scores_of_any_size_rank_the_same(M, N, k, B, policy):
    """Log-probabilities or raw scores instead of probabilities: values far below zero, infinities of either sign and the
    lowest double, in which nothing that pads a row or marks an expert outside the shortlist may take part."""
    print(f"case M={M} N={N} k={k} B={B} policy={policy}", flush=True)
    r = np.random.default_rng(M + N)
    g = r.integers(-(1 << 15), 1 << 12, size=(M, N)).astype(np.float64) / (1 << 12)
    g[:, r.permutation(N)[: N // 3]] -= 64.0
    g[r.integers(0, M, M), r.integers(0, N - 1, M)] = -np.inf
    g[r.integers(0, M, M // 2 + 1), r.integers(0, N - 1, M // 2 + 1)] = np.finfo(np.float64).min
    g[r.integers(0, M), N - 1] = np.inf
    desc = mb.LayerDesc(32, N, k, 32, mb.BF16, False)
    b = mb.moespec_budget(desc, torch.from_numpy(g).cuda(), B, policy, mb.alloc_workspace(desc, M))
    torch.cuda.synchronize()
    ids = np.array([O.top_k(row, k) for row in g], dtype=np.int32)
    w = np.array([O.mixing_weights(row, i, False) for row, i in zip(g, ids)])
    with np.errstate(over="ignore"):
        ref = O.budget(g, ids, w, B, policy, k, False)
        got = {key: val.cpu().numpy() for key, val in b.items()}
        assert np.array_equal(got["scores"], ref["scores"])
        assert np.array_equal(got["budget_ids"], ref["S"])
        assert np.array_equal(got["tok_ids"], ref["tok_ids"])
        assert np.array_equal(got["seg_expert"], ref["seg_expert"])
        assert np.array_equal(got["seg_off"], ref["seg_off"])
        assert np.array_equal(got["tok_w"], ref["tok_w"].astype(np.float32))


def best_us(N, M):
    """Time of one budget stage on the GPU: replayed 20 times from a graph, so that the host's calls do not count."""
    desc = mb.LayerDesc(512, N, 8, 32, mb.BF16, True)
    ws = mb.alloc_workspace(desc, M)
    probs = torch.softmax(torch.randn(M, N, dtype=torch.float64, device="cuda"), dim=1)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        mb.moespec_budget(desc, probs, N // 2, mb.SUBSTITUTE, ws)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(20):
            mb.moespec_budget(desc, probs, N // 2, mb.SUBSTITUTE, ws)
    times = []
    for _ in range(8):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        graph.replay()
        end.record()
        end.synchronize()
        times.append(start.elapsed_time(end) * 50.0)
    return min(times)


def test_one_expert_more_than_a_wave_per_token_takes_costs_no_multiple():
    """The selection has another form above 256 experts; 300 of them may cost the square of the ratio and the other form's
    overhead, not the eleven times that a wave with 16 candidates per lane took (63 tokens: 405 us against 37)."""
    few, many = best_us(256, 63), best_us(300, 63)
    print(f"256 experts {few:.1f} us, 300 experts {many:.1f} us", flush=True)
    assert many < 4 * few


def test_a_small_tree_does_not_queue_its_tokens_on_a_few_compute_units():
    """63 tokens x 256 experts at 16 waves per workgroup would be four workgroups (37 us for the stage against 12 for 64
    experts); with a workgroup per token the N^2 comparisons of the shortlist are the difference (17 us)."""
    few, many = best_us(64, 63), best_us(256, 63)
    print(f"64 experts {few:.1f} us, 256 experts {many:.1f} us", flush=True)
    assert many < 2.2 * few


@pytest.mark.parametrize("M,N,launches", [(128, 64, 2), (129, 64, 2), (256, 128, 2), (257, 64, 3), (129, 129, 3)])
def test_launches_of_a_budget_stage(M, N, launches):
    """The rows are summed by a launch of its own only where that is cheaper: a caller pays the host's share of each."""
    desc = mb.LayerDesc(32, N, 1, 32, mb.BF16, True)
    ws, probs = mb.alloc_workspace(desc, M), torch.rand(M, N, dtype=torch.float64, device="cuda")
    mb.moespec_budget(desc, probs, 1, mb.SUBSTITUTE, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        mb.moespec_budget(desc, probs, 1, mb.SUBSTITUTE, ws)
    n = ctypes.c_size_t()
    assert ctypes.CDLL("libamdhip64.so").hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    assert n.value == launches
