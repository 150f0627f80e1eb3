"""The calls whose speed is tracked: budgeted MoE-layer work over the sizes, types and options that programs use.

Four kinds of call, each through the binding's public entry points:

  layer      one layer forward on a draft tree (LayerForwardCall, what a verification loop keeps per layer)
  stack      consecutive layers joined by the residual stream (StackForwardCall)
  stages     route, budget and expert networks called one by one, with every table handed out
  calibrate  routing of a batch of calibration tokens, selection counts, static shortlist

Inputs follow the synthetic workloads of the package: hidden rows N(0, 1), weights N(0, 0.02), a router bias
alpha * log(1 / rank) with a seeded rank permutation that concentrates the routing on a few experts.
"""
import math

import torch

from paper_2602_16052_amd import binding as mb

SIGMA_W = 0.02
_DTYPE = {"bf16": (mb.BF16, torch.bfloat16, 2), "f32": (mb.F32, torch.float32, 4)}


def _layer(name, dtype, d, N, k, F, M, B, policy, renorm=True, alpha=1.5, gate="softmax", residual=False):
    return dict(name=name, kind="layer", dtype=dtype, d=d, N=N, k=k, F=F, M=M, B=B, policy=policy, renorm=renorm,
                alpha=alpha, gate=gate, residual=residual)


def listed():
    return [
        # the smallest layer in use: an fp32 block of a toy or draft model, 15-token tree; launches and latency count
        _layer("f32_tiny_m15", "f32", 128, 8, 2, 256, 15, 4, "substitute"),
        # fp32 in earnest: a small model verified at full precision, truncation on top of the residual stream
        _layer("f32_m63", "f32", 512, 16, 4, 1024, 63, 8, "truncate", residual=True),
        # 64 small experts, shortest useful draft (a chain of 7), tight budget
        _layer("olmoe_m7_b16", "bf16", 2048, 64, 8, 1024, 7, 16, "truncate", residual=True),
        # the benchmark's layer: default 63-token tree at half the experts
        _layer("olmoe_m63_b32", "bf16", 2048, 64, 8, 1024, 63, 32, "substitute"),
        # a wider tree under sigmoid gating, generous budget
        _layer("olmoe_m127_b48_sigmoid", "bf16", 2048, 64, 8, 1024, 127, 48, "truncate", gate="sigmoid", residual=True),
        # the upper end of the tree sizes
        _layer("olmoe_m511_b32", "bf16", 2048, 64, 8, 1024, 511, 32, "substitute"),
        # 128 experts, raw mixing weights
        _layer("fine_m127_b64", "bf16", 2048, 128, 8, 768, 127, 64, "substitute", renorm=False, alpha=1.2),
        # one rank's quarter of the same layer when the expert width is sharded over four GPUs: an odd width (192)
        _layer("fine_shard192_m127_b64", "bf16", 2048, 128, 8, 192, 127, 64, "substitute", renorm=False, alpha=1.2),
        # a prompt chunk through the same layer without a budget (B = N)
        _layer("olmoe_prefill_m2048", "bf16", 2048, 64, 8, 1024, 2048, 64, "truncate"),
        # whole call: four layers of 8 large experts at the tightest budget, B = k.  Every token then uses the whole
        # shortlist; with more candidates a near-tie that a rounding of the residual stream turns over swaps an
        # expert of one token, and that says nothing about precision
        dict(name="coarse_stack4_m63_b2", kind="stack", dtype="bf16", d=4096, N=8, k=2, F=14336, M=63, B=2,
             policy="substitute", renorm=True, alpha=1.5, gate="softmax", n_layers=4),
        # the stage calls of a program that looks at the routing tables (profiling, custom budgets)
        dict(name="stages_olmoe_m63_b32", kind="stages", dtype="bf16", d=2048, N=64, k=8, F=1024, M=63, B=32,
             policy="substitute", renorm=True, alpha=1.5, gate="softmax"),
        # static ranking: one batch of calibration tokens
        dict(name="calibrate_olmoe_m4096", kind="calibrate", dtype="bf16", d=2048, N=64, k=8, F=1024, M=4096, B=32,
             policy="substitute", renorm=True, alpha=1.5, gate="softmax"),
    ]


def _log_int(rng, lo, hi, mult=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / mult)) * mult))


def draw(rng):
    kind = rng.choice(["layer"] * 9 + ["f32"] * 3 + ["prefill", "stages", "stack", "calibrate"])
    dtype = "bf16"
    if kind == "f32":
        dtype, d, F = "f32", _log_int(rng, 64, 1024, 4), _log_int(rng, 64, 1024, 4)
        N, M = _log_int(rng, 4, 32), _log_int(rng, 1, 127)
    elif kind == "stack":
        d, F, N, M = _log_int(rng, 1024, 4096, 64), _log_int(rng, 1024, 8192, 64), rng.randint(4, 8), _log_int(rng, 1, 127)
    else:
        unit = rng.choice([32, 128])  # odd multiples of 32 are rank slices and narrow models
        d, F, N = _log_int(rng, 512, 4096, unit), _log_int(rng, 128, 2048, unit), _log_int(rng, 8, 128)
        while N * d * F > 3 << 27:
            F, N = max(128, F // 2 // unit * unit), max(8, N * 3 // 4)
        M = _log_int(rng, 512, 2048) if kind == "prefill" else _log_int(rng, 512, 4096) if kind == "calibrate" else _log_int(rng, 1, 511)
    k = min(N, rng.choice([1, 2, 4, 6, 8]))
    B = N if kind == "prefill" else k if kind == "stack" else rng.randint(k, N)
    case = dict(kind="layer" if kind in ("f32", "prefill") else kind, dtype=dtype, d=d, N=N, k=k, F=F, M=M, B=B,
                policy=rng.choice(["truncate", "substitute"]), renorm=rng.random() < 0.6,
                alpha=round(rng.uniform(0.5, 1.8), 2), gate="sigmoid" if rng.random() < 0.2 else "softmax")
    if kind == "stack":
        case["policy"] = "substitute"
        case["n_layers"] = rng.randint(2, 3)
    elif case["kind"] == "layer":
        case["residual"] = rng.random() < 0.4
    return case


def _desc(c):
    return mb.LayerDesc(c["d"], c["N"], c["k"], c["F"], _DTYPE[c["dtype"]][0], c["renorm"],
                        mb.GATE_SIGMOID if c["gate"] == "sigmoid" else mb.GATE_SOFTMAX)


def _bias(c, gen, device):
    rank = torch.randperm(c["N"], generator=gen, device=device) + 1
    return (c["alpha"] * torch.log(1.0 / rank.double())).float()


def _inputs(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    dt = _DTYPE[c["dtype"]][1]
    d, N, F, M = c["d"], c["N"], c["F"], c["M"]

    def normal(*shape, sigma=1.0):
        return torch.empty(shape, dtype=dt, device="cuda").normal_(0.0, sigma, generator=gen)

    layers = []
    for _ in range(c.get("n_layers", 1)):
        w = dict(w_router=normal(N, d, sigma=SIGMA_W), b_router=_bias(c, gen, "cuda"))
        if c["kind"] != "calibrate":
            w.update(w_gate=normal(N, F, d, sigma=SIGMA_W), w_up=normal(N, F, d, sigma=SIGMA_W),
                     w_down=normal(N, d, F, sigma=SIGMA_W))
        layers.append(w)
    return dict(layers=layers, h=normal(M, d), residual=normal(M, d) if c.get("residual") else None)


def prepare(case, seed):
    c, s = case, _inputs(case, seed)
    desc = _desc(c)
    policy = mb.TRUNCATE if c["policy"] == "truncate" else mb.SUBSTITUTE
    s.update(case=c, desc=desc, policy=policy, ws=mb.alloc_workspace(desc, c["M"]))
    if c["kind"] == "layer":
        s["out"] = torch.empty_like(s["h"])
        s["call"] = mb.LayerForwardCall(desc, s["layers"][0], s["h"], c["B"], policy, s["ws"], s["out"],
                                        residual=s["residual"])
    elif c["kind"] == "stack":
        s["stream"] = torch.empty_like(s["h"])
        s["call"] = mb.StackForwardCall(desc, s["layers"], s["stream"], c["B"], policy, s["ws"])
    return s


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "layer":
        s["call"]()
        return s["out"]
    if c["kind"] == "stack":
        s["stream"].copy_(s["h"])  # the hidden state comes from the model's embedding; the call updates it in place
        s["call"]()
        return s["stream"]
    desc, w, h, ws = s["desc"], s["layers"][0], s["h"], s["ws"]
    r = mb.moespec_route(desc, w, h, ws)
    if c["kind"] == "calibrate":
        counts = torch.zeros(c["N"], dtype=torch.int64, device=h.device)
        mb.moespec_calibration_count(desc, r["topk_ids"], counts)
        return dict(r, counts=counts, shortlist=mb.moespec_static_shortlist(desc, counts, c["B"]))
    b = mb.moespec_budget(desc, r["probs"], c["B"], s["policy"], ws)
    out = mb.moespec_expert_ffn(desc, w, h, b["seg_expert"], b["seg_off"], b["perm"], b["tok_ids"], b["tok_w"], ws)
    return dict(route=r, budget=b, out=out)


# ---- the same in 64 bits, plain torch ---------------------------------------------------------------------------
def _top(v, k):
    """ids of the k largest per row, ties to the lowest id"""
    return torch.sort(v, dim=-1, descending=True, stable=True).indices[..., :k]


def _probabilities(c, logits):
    return torch.sigmoid(logits) if c["gate"] == "sigmoid" else torch.softmax(logits, dim=-1)


def _weights_of(c, g, ids):
    w = g.gather(1, ids)
    return w / w.sum(1, keepdim=True) if c["renorm"] else w


def _restrict(c, g):
    """(shortlist, ids [M, k] with -1 for dropped slots, weights) from the routing probabilities"""
    S = _top(g.sum(0), c["B"])
    inside = torch.zeros(c["N"], dtype=torch.bool, device=g.device)
    inside[S] = True
    if c["policy"] == "truncate":
        ids = _top(g, c["k"])
        w, keep = _weights_of(c, g, ids), inside[ids]
        return S, torch.where(keep, ids, -1), torch.where(keep, w, 0.0)
    ids = _top(torch.where(inside, g, -1.0), c["k"])
    return S, ids, _weights_of(c, g, ids)


def _experts(c, w, x, ids, wt):
    out = torch.zeros(x.shape, dtype=torch.float64, device=x.device)
    for e in sorted(set(ids.flatten().tolist()) - {-1}):
        t, slot = (ids == e).nonzero(as_tuple=True)
        xe = x[t].double()
        a = torch.nn.functional.silu(xe @ w["w_gate"][e].double().t()) * (xe @ w["w_up"][e].double().t())
        out.index_add_(0, t, wt[t, slot].unsqueeze(1) * (a @ w["w_down"][e].double().t()))
    return out


def _route64(c, w, x):
    return _probabilities(c, x.double() @ w["w_router"].double().t() + w["b_router"].double())


def exact(case, seed):
    c, s = case, _inputs(case, seed)
    w, h, dt = s["layers"][0], s["h"], _DTYPE[case["dtype"]][1]
    if c["kind"] == "stack":
        # the residual stream and the scaled layer inputs are stored in the layer's type between layers
        for w in s["layers"]:
            x = h.double()
            x = (x / x.square().mean(1, keepdim=True).sqrt()).to(dt)
            _, ids, wt = _restrict(c, _route64(c, w, x))
            last = h.double() + _experts(c, w, x, ids, wt)
            h = last.to(dt)
        return last
    g = _route64(c, w, h)
    if c["kind"] == "layer":
        _, ids, wt = _restrict(c, g)
        out = _experts(c, w, h, ids, wt)
        return out + s["residual"].double() if s["residual"] is not None else out
    top = _top(g, c["k"])
    r = dict(probs=g, topk_ids=top.int(), topk_w=_weights_of(c, g, top))
    if c["kind"] == "calibrate":
        counts = torch.bincount(top.flatten(), minlength=c["N"])
        return dict(r, counts=counts, shortlist=_top(counts, c["B"]).int())
    S, ids, wt = _restrict(c, g)
    seg = torch.sort(S).values
    pairs = [((ids == e).nonzero(as_tuple=True)) for e in seg.tolist()]
    flat = [t * c["k"] + slot for t, slot in pairs]
    sizes = torch.tensor([0] + [p.numel() for p in flat], device=h.device)
    perm = torch.full((c["M"] * c["k"],), -1, dtype=torch.int32, device=h.device)
    perm[: int(sizes.sum())] = torch.cat(flat).int()
    b = dict(scores=g.sum(0), budget_ids=S.int(), tok_ids=ids.int(), tok_w=wt, seg_expert=seg.int(),
             seg_off=torch.cumsum(sizes, 0).int(), perm=perm, n_loaded=(sizes[1:] > 0).sum().reshape(1).int())
    return dict(route=r, budget=b, out=_experts(c, w, h, ids, wt))


def work(case):
    """Bytes: the loaded experts, the router, the hidden rows in and out, the tables a caller gets.  The number of
    loaded experts and of surviving pairs is that of one draw of router logits with the case's distribution."""
    c = case
    es = _DTYPE[c["dtype"]][2]
    d, N, k, F, M, L = c["d"], c["N"], c["k"], c["F"], c["M"], c.get("n_layers", 1)
    gen = torch.Generator().manual_seed(1)
    logits = torch.randn(M, N, generator=gen, dtype=torch.float64) * (SIGMA_W * math.sqrt(d)) + _bias(c, gen, "cpu").double()
    _, ids, _ = _restrict(c, _probabilities(c, logits))
    loaded, pairs = len(set(ids.flatten().tolist()) - {-1}), int((ids >= 0).sum())
    bytes_, flops = N * d * es + M * d * es, 2 * M * N * d
    if c["kind"] in ("stages", "calibrate"):
        bytes_ += M * N * 8 + M * k * 8  # probabilities and the natural top-k
    if c["kind"] != "calibrate":
        bytes_ += loaded * 3 * d * F * es + M * d * es * (2 if c.get("residual") else 1)
        flops += 6 * d * F * pairs
    return {"bytes": bytes_ * L, "flops": flops * L}


def tolerance(case):
    """About four times the measured error of the path against exact(), which bounds what another order of the sums
    does: 2.3e-3 for one bf16 layer (act and out are stored in bf16), 7e-3 for four layers of a stack, 1.6e-7 in
    fp32, 3e-8 for weights that are stored in fp32."""
    if case["kind"] == "calibrate":
        return {"rel": 1e-7}
    if case["kind"] == "stack":
        return {"rel": 3e-2}
    return {"rel": 1e-2 if case["dtype"] == "bf16" else 8e-7}
