"""The work a user of this framework has it do, as cases to time and to compare.

Six kinds of pass, each through the public entry points of the package:

  step   one training step of the output layer as one call that selects its own batch's classes
         (knn_softmax_fwd_bwd_update), or as two calls where the caller wants the weight gradient
         (knn_softmax_fwd_bwd, apply_weight_grad)
  loop   a training loop's step: forward, backward and update of this batch, selection of the next one inside the same
         call (knn_softmax_fwd_bwd_update_selected_next); either with the plain update, or as a layer that owns the
         normalisation of X and W (knn_normalize_rows, knn_norm_backward_rows, apply_weight_grad_normalized)
  node   one node of the sharded layer: statistics out, statistics of all nodes in, gradients, normalised update, the
         next batch's selection on the node's compressed graph
  graph  the periodic exact rebuild of the class graph on one GPU
  ring   one node's part of the distributed rebuild: every shard of W visits once
  topk   exact layer-wise top-k selection over a model's gradient tensors

Sizes are those of the repository's configurations (10,000 to 1,000,000 classes, D 64 to 512, batches 64 to 2,048).
Inputs are made on the GPU from the seed alone.
"""
import math
import random

import torch

import paper_2102_06025_amd as ks

SCALE, GRAD_SCALE, LR = 30.0, 128.0, 0.05
ALPHA = -LR / GRAD_SCALE
MAX_WORK = 2048 * 131_072 * 512  # B * active classes * D of the largest listed step
MAX_PAIRS = 390_625 * 390_625 * 512  # C * C * D of the largest listed rebuild


# ---------------------------------------------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest steps: launches and host time count
        {"name": "step_tiny", "kind": "step", "C": 10_000, "D": 128, "B": 64, "K": 8, "M": 1_024, "labels": "uniform",
         "unit": True, "fused": True},
        # a small problem on which the cut to M classes bites
        {"name": "step_small", "kind": "step", "C": 100_000, "D": 256, "B": 256, "K": 16, "M": 4_096, "labels": "uniform",
         "unit": True, "fused": True},
        # an odd-sized problem of a caller with rows of any norm and an optimiser of its own: the gradient rows come out
        {"name": "step_ragged", "kind": "step", "C": 50_021, "D": 320, "B": 333, "K": 12, "M": 3_001, "labels": "zipf",
         "unit": False, "fused": False},
        # one GPU's share of 100 M classes, rows of any norm (two-sweep softmax)
        {"name": "step_shard_general", "kind": "step", "C": 390_625, "D": 512, "B": 1_024, "K": 32, "M": 32_768,
         "labels": "zipf", "unit": False, "fused": True},
        # a million classes on one GPU: the largest step
        {"name": "step_million", "kind": "step", "C": 1_000_000, "D": 512, "B": 2_048, "K": 64, "M": 131_072,
         "labels": "uniform", "unit": True, "fused": True},
        # the benchmark's training loop
        {"name": "loop_shard", "kind": "loop", "C": 390_625, "D": 512, "B": 1_024, "K": 32, "M": 32_768, "labels": "zipf",
         "normalised": False},
        # the same shard with labels that fill the active set, and the normalisation inside the layer
        {"name": "layer_shard_cap", "kind": "loop", "C": 390_625, "D": 512, "B": 1_024, "K": 32, "M": 32_768,
         "labels": "uniform", "normalised": True},
        # one of four nodes of a sharded layer
        {"name": "node_of_four", "kind": "node", "C": 390_625, "nodes": 4, "D": 512, "B": 1_024, "K": 32, "M": 32_768,
         "labels": "zipf", "fill": False},
        # graph rebuild of a small problem from fp32 weights
        {"name": "graph_small", "kind": "graph", "C": 10_000, "D": 128, "K": 8, "bf16": False, "clustered": False},
        # graph rebuild of the shard
        {"name": "graph_shard", "kind": "graph", "C": 390_625, "D": 512, "K": 32, "bf16": True, "clustered": False},
        # the distributed rebuild of a small problem over four nodes
        {"name": "ring_of_four", "kind": "ring", "C": 100_000, "nodes": 4, "D": 256, "K": 16, "bf16": True},
        # the gradient tensors of a ResNet-50, 99.9 % sparsity
        {"name": "topk_resnet50", "kind": "topk", "net": "resnet50", "tensors": 161, "largest": 2_359_296, "density": 0.001},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_layer(rng, kind):
    while True:
        C = _log(rng, 5_000, 1_000_000) if kind == "step" else _log(rng, 20_000, 500_000)
        D = rng.choice((64, 96, 128, 160, 256, 256, 320, 384, 512, 512)) if kind == "step" else rng.choice((128, 256, 512))
        B = _log(rng, 33, 2_048) if kind == "step" else rng.choice((_log(rng, 128, 2_048), 256, 512, 1_024))
        K = rng.choice((4, 8, 12, 16, 24, 32, 48, 64))
        # from a cut that bites to a cap that is never reached; a label and a whole list always fit
        M = int(B * (K + 1) * math.exp(rng.uniform(math.log(0.4), math.log(1.5))))
        M = max(B, K + 1, min(M, C, 131_072))
        if B * M * D <= MAX_WORK and (D % 64 == 0 or B * M <= 1 << 25):
            break
    return {"C": C, "D": D, "B": B, "K": K, "M": M, "labels": rng.choice(("zipf", "uniform"))}


def draw(rng):
    kind = rng.choice(("step", "step", "step", "step", "loop", "loop", "node", "graph", "graph", "ring", "topk"))
    if kind == "topk":
        return {"kind": kind, "net": "", "tensors": rng.randint(3, 200), "largest": _log(rng, 20_000, 3_000_000),
                "density": rng.choice((0.0005, 0.001, 0.001, 0.002))}
    if kind == "graph":
        bf16 = rng.random() < 0.7
        while True:
            # fp32 weights: small problems; bf16 ones up to the shard
            C, D = _log(rng, 2_000, 390_625 if bf16 else 40_000), rng.choice((64, 128, 256, 320, 512))
            if C * C * D <= MAX_PAIRS // (1 if D in (128, 256, 512) else 4):
                break
        return {"kind": kind, "C": C, "D": D, "K": rng.choice((8, 16, 24, 32, 64)), "bf16": bf16,
                "clustered": bf16 and rng.random() < 0.3}
    if kind == "ring":
        return {"kind": kind, "C": _log(rng, 8_000, 150_000), "nodes": rng.choice((2, 3, 4)), "D": rng.choice((128, 256, 512)),
                "K": rng.choice((8, 16, 32)), "bf16": rng.random() < 0.75}
    case = {"kind": kind, **_draw_layer(rng, kind)}
    if kind == "step":
        case["unit"], case["fused"] = rng.random() < 0.75, rng.random() < 0.7
    elif kind == "loop":
        case["normalised"] = rng.random() < 0.5
    else:
        case["nodes"], case["fill"] = rng.choice((2, 4)), rng.random() < 0.4
    return case


# ---------------------------------------------------------------------------------------------------- inputs
def _rows(gen, n, D, clustered=False):
    """Rows of norm 1; clustered: 4,096 centres with noise of 0.3 of their norm."""
    W = torch.randn((n, D), generator=gen, device="cuda")
    if clustered:
        centres = torch.nn.functional.normalize(torch.randn((4096, D), generator=gen, device="cuda"))
        W = centres[torch.arange(n, device="cuda") % 4096] + W.mul_(0.3 / math.sqrt(D))
    return torch.nn.functional.normalize(W)


def _labels(gen, B, C, law):
    if law == "uniform":
        return torch.randint(0, C, (B,), generator=gen, device="cuda", dtype=torch.int32)
    # Zipf with exponent 1.1 over the ranks, ranks dealt to the classes at random
    cdf = torch.arange(1, C + 1, device="cuda", dtype=torch.float64).pow_(-1.1).cumsum_(0)
    u = torch.rand(B, generator=gen, device="cuda", dtype=torch.float64) * cdf[-1]
    rank = torch.searchsorted(cdf, u).clamp_(max=C - 1)
    return torch.randperm(C, generator=gen, device="cuda")[rank].to(torch.int32)


def _lists(gen, C, K):
    """K neighbour ids per class, none of them the class itself (the neighbours of random rows are random ids)."""
    c = torch.arange(C, device="cuda", dtype=torch.int64)[:, None]
    k = torch.arange(K, device="cuda", dtype=torch.int64)[None, :]
    first = torch.randint(0, C - 1, (C, 1), generator=gen, device="cuda", dtype=torch.int64)
    return ((c + 1 + (first + k * 40503) % (C - 1)) % C).to(torch.int32)


def _features(gen, W, rows, B, D):
    """Features of a half-trained model: between a random direction and the class's own weight."""
    X = torch.nn.functional.normalize(torch.randn((B, D), generator=gen, device="cuda"))
    near = torch.rand((B, 1), generator=gen, device="cuda") * 0.6
    own = (rows >= 0)[:, None]
    X = torch.where(own, X * (1 - near) + W[rows.clamp(min=0).long()] * near, X)
    return torch.nn.functional.normalize(X)


def _f32(*shape):
    return torch.zeros(shape, dtype=torch.float32, device="cuda")


def _i32(n):
    return torch.zeros(n, dtype=torch.int32, device="cuda")


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def _sizes(case):
    """Element counts of the case's gradient tensors."""
    if case["net"] == "resnet50":  # convolutions, scale and shift after each, classifier
        sizes, width = [64 * 3 * 49, 64, 64], 64
        for p, blocks in ((64, 3), (128, 4), (256, 6), (512, 3)):
            for b in range(blocks):
                sizes += [p * width, p, p, 9 * p * p, p, p, 4 * p * p, 4 * p, 4 * p]
                if b == 0:
                    sizes += [4 * p * width, 4 * p, 4 * p]
                width = 4 * p
        return sizes + [2048 * 1000, 1000]
    r = random.Random(case["tensors"] * 7919 + case["largest"])
    sizes = [_log(r, 64, case["largest"]) for _ in range(case["tensors"])]
    sizes[r.randrange(len(sizes))] = case["largest"]
    return sizes


def _k(n, density):
    return max(1, min(4096, int(n * density)))


def _prepare_step(case, gen):
    C, D, B, K, M = (case[k] for k in ("C", "D", "B", "K", "M"))
    W = _rows(gen, C, D)
    y = _labels(gen, B, C, case["labels"])
    X = _features(gen, W, y, B, D).to(torch.bfloat16)
    out = {"active_idx": _i32(M), "n_active": _i32(1), "target_pos": _i32(B), "loss_per_sample": _f32(B), "loss_mean": _f32(1),
           "dX": _f32(B, D), "dW_active": None if case["fused"] and D % 64 == 0 else _f32(M, D), "dev_status": _i32(1)}
    s = {"W": W, "Wb": W.to(torch.bfloat16), "X": X, "labels": y, "lists": _lists(gen, C, K), "out": out,
         "ws": _bytes(ks.knn_softmax_workspace(C, D, B, K, M))}
    if not case["fused"]:
        s["apply_ws"] = _bytes(ks.apply_weight_grad_workspace(C, D, M, True))
    return s


def _run_step(s):
    c, o = s["case"], s["out"]
    if c["fused"]:
        ks.knn_softmax_fwd_bwd_update(s["W"], s["Wb"], s["X"], s["labels"], s["lists"], c["M"], SCALE, GRAD_SCALE, ALPHA, out=o,
                                      ws=s["ws"], unit_rows=c["unit"])
        grad = []
    else:
        ks.knn_softmax_fwd_bwd(s["Wb"], s["X"], s["labels"], s["lists"], c["M"], SCALE, GRAD_SCALE, out=o, ws=s["ws"],
                               unit_rows=c["unit"])
        ks.apply_weight_grad(s["W"], s["Wb"], o["active_idx"], o["n_active"], o["dW_active"], ALPHA, idx_sorted_unique=True,
                             ws=s["apply_ws"], dev_status=o["dev_status"])
        grad = [o["dW_active"]]
    return [o["active_idx"], o["n_active"], o["target_pos"], o["loss_per_sample"], o["loss_mean"], o["dX"], o["dev_status"],
            s["W"], s["Wb"]] + grad


def _prepare_loop(case, gen):
    C, D, B, K, M = (case[k] for k in ("C", "D", "B", "K", "M"))
    W = _rows(gen, C, D)
    s = {"W": W, "lists": _lists(gen, C, K), "turn": 0, "status": _i32(1)}
    s["labels"] = [_labels(gen, B, C, case["labels"]) for _ in range(2)]
    X = [_features(gen, W, y, B, D) for y in s["labels"]]
    if case["normalised"]:  # weights and features of any norm, the layer keeps the normalised copy and the inverse norms
        W.mul_(0.5 + torch.rand((C, 1), generator=gen, device="cuda"))
        s["Wb"], s["inv"] = ks.knn_normalize_rows(W)
        s["X"] = [x * (5 + 10 * torch.rand((B, 1), generator=gen, device="cuda")) for x in X]
        s["Xb"], s["dx"] = torch.empty((B, D), dtype=torch.bfloat16, device="cuda"), _f32(B, D)
        s["apply_ws"] = _bytes(ks.apply_weight_grad_normalized_workspace(C, D, M, True))
    else:
        s["Wb"] = W.to(torch.bfloat16)
        s["X"] = [x.to(torch.bfloat16) for x in X]
    s["out"] = {"loss_per_sample": _f32(B), "loss_mean": _f32(1), "dX": _f32(B, D),
                "dW_active": _f32(M, D) if case["normalised"] else None, "dev_status": s["status"]}
    s["ws"] = _bytes(ks.knn_softmax_selected_next_workspace(C, D, B, K, M))
    idx, n, pos, _ = ks.knn_select_active(s["labels"][0], s["lists"], C, M)
    s["sel"] = [{"active_idx": idx, "n_active": n, "target_pos": pos},
                {"active_idx": _i32(M), "n_active": _i32(1), "target_pos": _i32(B)}]
    return s


def _run_loop(s):
    c, o, t = s["case"], s["out"], s["turn"]
    here, then, X = s["sel"][t], s["sel"][1 - t], s["X"][t]
    norm = c["normalised"]
    if norm:
        ks.knn_normalize_rows(X, want_inv_norm=False, out_bf16=s["Xb"])
    ks.knn_softmax_fwd_bwd_update_selected_next(None if norm else s["W"], s["Wb"], s["Xb"] if norm else X, here["active_idx"],
                                                here["n_active"], here["target_pos"], s["labels"][1 - t], s["lists"], SCALE,
                                                GRAD_SCALE, ALPHA, next_out=then, out=o, ws=s["ws"], unit_rows=True,
                                                trusted_list=True)
    s["turn"] = 1 - t
    got = [o["loss_per_sample"], o["loss_mean"], o["dX"], then["active_idx"], then["n_active"], then["target_pos"], s["status"],
           s["W"], s["Wb"]]
    if norm:
        ks.knn_norm_backward_rows(X, o["dX"], out=s["dx"])
        ks.apply_weight_grad_normalized(s["W"], s["Wb"], s["inv"], here["active_idx"], here["n_active"], o["dW_active"], ALPHA,
                                        idx_sorted_unique=True, ws=s["apply_ws"], dev_status=s["status"])
        got += [s["dx"], s["inv"], o["dW_active"]]
    return got


def _prepare_node(case, gen):
    C, D, B, K, M, P = (case[k] for k in ("C", "D", "B", "K", "M", "nodes"))
    Cg, c0 = P * C, C
    W = _rows(gen, C, D)
    s = {"turn": 0, "status": _i32(1), "c0": c0}
    s["labels"] = [_labels(gen, B, Cg, case["labels"]) for _ in range(2)]
    s["X"] = []
    for y in s["labels"]:
        local = y - c0
        X = _features(gen, W, torch.where((local >= 0) & (local < C), local, -1), B, D)
        s["X"].append(X * (5 + 10 * torch.rand((B, 1), generator=gen, device="cuda")))
    lists = _lists(gen, Cg, K)
    s["csr"] = ks.knn_graph_compress(lists, c0, C)[:3]
    del lists
    s["W"] = W.mul_(0.5 + torch.rand((C, 1), generator=gen, device="cuda"))
    s["Wb"], s["inv"] = ks.knn_normalize_rows(W)
    s["Xb"] = torch.empty((B, D), dtype=torch.bfloat16, device="cuda")
    # what the other nodes' sums and target logits come to
    s["sum"] = (P - 1) * (1000 + 200 * torch.rand(B, generator=gen, device="cuda")) * math.exp(-SCALE)
    s["tz"] = [torch.where((y >= c0) & (y < c0 + C), 0.0, SCALE / math.sqrt(D) * torch.randn(B, generator=gen, device="cuda"))
               for y in s["labels"]]
    s["stats"] = {"row_max": _f32(B), "row_sumexp": _f32(B), "target_logit": _f32(B)}
    s["out"] = {"loss_per_sample": _f32(B), "loss_mean": _f32(1), "dX": _f32(B, D), "dW_active": _f32(M, D), "dev_status": s["status"]}
    s["ws"] = _bytes(ks.knn_softmax_split_next_workspace(C, D, B, K, M))
    s["apply_ws"] = _bytes(ks.apply_weight_grad_normalized_workspace(C, D, M, True))
    first = ks.knn_select_active_csr(s["labels"][0], *s["csr"], c0, C, K, M, pad_random=case["fill"], pad_seed=1)
    s["sel"] = [{k: first[k] for k in ("active_idx", "n_active", "n_found", "target_pos")},
                {"active_idx": _i32(M), "n_active": _i32(1), "n_found": _i32(1), "target_pos": _i32(B)}]
    return s


def _run_node(s):
    c, o, t, st = s["case"], s["out"], s["turn"], s["stats"]
    here, then = s["sel"][t], s["sel"][1 - t]
    ks.knn_normalize_rows(s["X"][t], want_inv_norm=False, out_bf16=s["Xb"])
    ks.knn_softmax_fwd_stats(s["Wb"], s["Xb"], here["active_idx"], here["n_active"], here["target_pos"], SCALE, unit_rows=True,
                             ws=s["ws"], dev_status=s["status"], trusted_list=True, out=st)
    # the all-reduce over the nodes: with unit rows the sums and the target logits just add up
    st["row_sumexp"] += s["sum"]
    st["target_logit"] += s["tz"][t]
    ks.knn_softmax_bwd_from_stats_next(s["Wb"], s["Xb"], here["active_idx"], here["n_active"], here["target_pos"], st["row_max"],
                                       st["row_sumexp"], st["target_logit"], SCALE, GRAD_SCALE, s["ws"], s["labels"][1 - t],
                                       *s["csr"], s["c0"], c["K"], next_out=then, pad_random=c["fill"], pad_seed=2 + t,
                                       unit_rows=True, trusted_list=True, dev_status=s["status"], out=o)
    ks.apply_weight_grad_normalized(s["W"], s["Wb"], s["inv"], here["active_idx"], here["n_active"], o["dW_active"], ALPHA,
                                    idx_sorted_unique=True, ws=s["apply_ws"], dev_status=s["status"])
    s["turn"] = 1 - t
    return [o["loss_per_sample"], o["loss_mean"], o["dX"], o["dW_active"], then["active_idx"], then["n_active"], then["n_found"],
            then["target_pos"], s["status"], s["W"], s["Wb"], s["inv"]]


def _prepare_graph(case, gen):
    C, D, K = case["C"], case["D"], case["K"]
    W = _rows(gen, C, D, case["clustered"])
    if case["bf16"]:
        W = W.to(torch.bfloat16)
    return {"W": W, "graph": torch.empty((C, K), dtype=torch.int32, device="cuda"), "sims": _f32(C, K), "status": _i32(1),
            "ws": _bytes(ks.knn_graph_build_workspace(C, D, K, 0 if case["bf16"] else 1))}


def _run_graph(s):
    ks.knn_graph_build(s["W"], s["case"]["K"], want_sims=True, graph=s["graph"], sims=s["sims"], ws=s["ws"], dev_status=s["status"])
    return [s["graph"], s["sims"], s["status"]]


def _prepare_ring(case, gen):
    C, D, K, P = (case[k] for k in ("C", "D", "K", "nodes"))
    W = _rows(gen, C, D)
    if case["bf16"]:
        W = W.to(torch.bfloat16)
    bounds = [C * p // P for p in range(P + 1)]
    shards = [(lo, W[lo:hi].clone()) for lo, hi in zip(bounds, bounds[1:])]
    n, most = bounds[1], max(hi - lo for lo, hi in zip(bounds, bounds[1:]))
    return {"shards": shards, "graph": torch.empty((n, K), dtype=torch.int32, device="cuda"),
            "sims": torch.empty((n, K), dtype=torch.float64, device="cuda"), "status": _i32(1),
            "ws": _bytes(ks.knn_graph_update_workspace(n, most, D, K, 0 if case["bf16"] else 1))}


def _run_ring(s):
    s["graph"].fill_(-1)
    s["sims"].fill_(-math.inf)
    for lo, visit in s["shards"]:
        ks.knn_graph_update(s["shards"][0][1], visit, 0, lo, s["graph"], s["sims"], ws=s["ws"], dev_status=s["status"])
    return [s["graph"], s["sims"], s["status"]]


def _prepare_topk(case, gen):
    sizes = _sizes(case)
    offsets = [0]
    for n in sizes:
        offsets.append(offsets[-1] + n)
    g = torch.randn(offsets[-1], generator=gen, device="cuda")
    for t, n in enumerate(sizes):  # layers of different scale; in every fifth one dead units and repeated values
        part = g[offsets[t]:offsets[t + 1]]
        part.mul_(1e-3 * 2.0 ** (t % 7 - 3))
        if t % 5 == 0 and n >= 8:
            e, q = n // 8, 2.5e-4 * 2.0 ** (t % 7 - 3)
            part[e:2 * e] = 0
            part[2 * e:3 * e] = (part[2 * e:3 * e] / q).round_().mul_(q)
    plan = ks.grad_topk_plan(offsets, [_k(n, case["density"]) for n in sizes])
    return {"g": g, "plan": plan, "idx": _i32(plan.n_out), "val": _f32(plan.n_out), "ws": _bytes(plan.ws_bytes)}


def _run_topk(s):
    return list(ks.grad_topk_select(s["g"], s["plan"], out_idx=s["idx"], out_val=s["val"], ws=s["ws"]))


_PREPARE = {"step": _prepare_step, "loop": _prepare_loop, "node": _prepare_node, "graph": _prepare_graph, "ring": _prepare_ring,
            "topk": _prepare_topk}
_RUN = {"step": _run_step, "loop": _run_loop, "node": _run_node, "graph": _run_graph, "ring": _run_ring, "topk": _run_topk}


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    state = _PREPARE[case["kind"]](case, gen)
    state["case"] = case
    return state


def run(state):
    return _RUN[state["case"]["kind"]](state)


# ---------------------------------------------------------------------------------------------------- what it comes to
def _active(case):
    """Expected number of active classes (on this node)."""
    C, B, K, M = (case[k] for k in ("C", "B", "K", "M"))
    P = case.get("nodes", 1)
    if case.get("fill"):
        return min(M, C)
    Cg = P * C
    if case["labels"] == "uniform":
        distinct = Cg * -math.expm1(-B / Cg)
    else:
        total = sum(r ** -1.1 for r in range(1, 2001)) + (2000.5 ** -0.1 - (Cg + 0.5) ** -0.1) / 0.1
        distinct, r = 0.0, 1
        while r <= Cg:  # ranks in groups that grow by a thousandth
            n = min(max(1, r // 1000), Cg - r + 1)
            distinct += n * -math.expm1(-B * (r + (n - 1) / 2) ** -1.1 / total)
            r += n
    return min(M, C * -math.expm1(-distinct * (K + 1) / Cg))


def work(case):
    """bytes: inputs read once, outputs written once; flops: the contractions (a pair of rows of the graph counts once)."""
    kind = case["kind"]
    if kind == "topk":
        sizes = _sizes(case)
        return {"bytes": 4.0 * sum(sizes) + 8.0 * sum(_k(n, case["density"]) for n in sizes), "flops": 0.0}
    C, D, K = case["C"], case["D"], case["K"]
    if kind == "graph":
        return {"bytes": C * (D * (2.0 if case["bf16"] else 4.0) + K * 8.0), "flops": float(C) * (C - 1) * D}
    if kind == "ring":
        n = C // case["nodes"]
        return {"bytes": C * D * (2.0 if case["bf16"] else 4.0) + n * K * 12.0,
                "flops": 2.0 * n * (C - n) * D + float(n) * (n - 1) * D}
    A, B, M = _active(case), case["B"], case["M"]
    got = B * (8.0 + 4 * K + 4) + M * 4.0 + B * D * (2 + 4.0)  # labels, lists, target positions, losses, active list, X, dX
    rows = A * D * (2 + 4 + 4 + 2.0)  # 16-bit rows read and written, fp32 rows read and written
    if kind == "step" and not case["fused"] or kind == "node" or kind == "loop" and case["normalised"]:
        rows += A * D * 4.0  # the gradient rows are an output
    if kind == "loop" and case["normalised"]:
        got += B * D * (2 + 4.0)  # fp32 X, dX through the normalisation
    return {"bytes": got + rows, "flops": 6.0 * A * B * D}


def tolerance(case):
    """Whole numbers are exact everywhere; the softmax works on bf16 operands and stores its gradient in bf16."""
    return {"rel": 1e-2} if case["kind"] in ("step", "loop", "node") else "exact"
