"""The route stage where its dispatch changes: one slice or several of the hidden dimension (1024 / 1025 tokens),
experts around the candidates-per-lane steps and around the limit of the matrix-core projection, top-k of a whole wave;
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
                                          (5, 257, 8, 64, "softmax"), (2050, 1, 1, 32, "softmax")])
def test_route_stage_edges(M, N, k, d, gate):
    print(f"case M={M} N={N} k={k} d={d} {gate}", flush=True)
    cfg = wl.small_config("route_edge", "bf16", d=d, n_experts=N, top_k=k, d_ff=32, M=M, gate=gate, seed=M + N)
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
