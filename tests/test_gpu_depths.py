"""Problem depths and sizes at the edges of the kernels' dispatch: row lengths that are odd multiples of 32 or not a power of
two, searches cut into parts, and the sizes on both sides of the line between the two recall passes."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ks():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2102_06025_amd as ks
    ks.lib()
    return ks


def size_with_last_part(ks, n_loc, D, K, last):
    """The least number of visiting rows from 4,000 on for which the halves of a workgroup take turns and the last part is as wanted (None:
    not below 60,000)."""
    for n in range(4000, 60_000):
        p = ks.knn_graph_recall_plan(n_loc, n, D, K, 0)
        rows, whole = n - (p["parts"] - 1) * p["part_rows"], p["part_rows"] % p["chunk"] == 0
        if p["turns"] and {"one row": whole and rows == 1, "one chunk": whole and rows == p["chunk"], "no whole chunks": not whole,
                           "a chunk and some": whole and p["chunk"] < rows < 2 * p["chunk"]}[last]:
            return n
    return None


def dev(a, bf16=False):
    import torch
    t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    return t.to(torch.bfloat16) if bf16 else t


@pytest.mark.parametrize("C,D,K,bf16", [
    (31, 32, 5, True), (97, 64, 64, False), (300, 96, 33, True), (2049, 160, 16, False), (6143, 224, 32, True), (2500, 288, 17, True),
    (7001, 320, 64, True), (4097, 384, 8, False), (3001, 416, 32, True), (3500, 448, 16, True), (2300, 480, 48, False), (12_289, 192, 24, True),
    (29_296, 512, 32, True), (29_297, 512, 16, True), (58_594, 256, 8, True), (117_188, 128, 32, True)])
def test_graph_at_every_depth_and_around_the_symmetric_pass(ks, orc, C, D, K, bf16):
    """Fixed-threshold recall: depths of 1 to 8 k-tiles, whole and ragged; fewer rows than one sample, than one chunk, than one
    block; sizes of the pass that computes every similarity once (29,296 rows and more; its first sizes are in
    test_graph_around_the_smallest_symmetric_pass)."""
    import torch
    print(f"[depths] graph C={C} D={D} K={K} bf16={bf16}", flush=True)
    W = synth.unit_rows(21, synth.TID_W, C, D, bf16=bf16)
    W[C - 1] = W[C // 3]                                          # an exact twin
    rows = np.unique(np.concatenate([synth.class_permutation(21, C)[:120], [0, C // 3, C - 1], np.arange(max(0, C - 3), C)])).astype(np.int32)
    g, s = ks.knn_graph_build(dev(W, bf16), K, want_sims=True)
    torch.cuda.synchronize()
    eg, es = orc.graph_bruteforce(W, K, rows)
    assert (g.cpu().numpy()[rows] == eg).all() and (s.cpu().numpy()[rows] == es.astype(np.float32)).all()


@pytest.mark.parametrize("C_loc,C_vis,D,K,bf16", [(300, 20_011, 320, 16, True), (257, 9_000, 96, 64, False), (5000, 40, 512, 32, True),
                                                  (1, 6_001, 64, 32, True)])
def test_hop_cut_into_parts(ks, orc, C_loc, C_vis, D, K, bf16):
    """One hop of few local rows against many visiting ones (many parts), and the reverse; the shard visits twice (the second
    visit starts from full lists, or from short ones where the shard is smaller than K, and changes nothing)."""
    import torch
    print(f"[depths] hop {C_loc} x {C_vis} D={D} K={K} bf16={bf16}", flush=True)
    W = synth.unit_rows(22, synth.TID_W, C_loc + C_vis, D, bf16=bf16)
    Wl, Wv = dev(W[:C_loc], bf16), dev(W[C_loc:], bf16)
    graph = torch.full((C_loc, K), -1, dtype=torch.int32, device="cuda")
    sims = torch.full((C_loc, K), -np.inf, dtype=torch.float64, device="cuda")
    for _ in range(2):
        ks.knn_graph_update(Wl, Wv, 0, C_loc, graph, sims)
        torch.cuda.synchronize()
        S = W[:C_loc].astype(np.float64) @ W[C_loc:].astype(np.float64).T
        for i in (0, C_loc // 2, C_loc - 1):
            n = min(K, C_vis)
            best = np.argsort(-S[i], kind="stable")[:n] + C_loc
            got = graph[i].cpu().numpy()
            assert (got[:n] == best).all() and (got[n:] == -1).all()
            assert np.allclose(sims[i].cpu().numpy()[:n], S[i][best - C_loc], rtol=0, atol=1e-12)


@pytest.mark.parametrize("D", [32, 64, 96, 160, 192, 224, 256, 320, 352, 384, 448, 480, 512, 544, 576])
@pytest.mark.parametrize("C,B,K,M", [(700, 33, 6, 200), (3000, 300, 9, 2500)])
def test_step_at_every_depth(ks, orc, D, C, B, K, M):
    """Forward and backward in both softmax modes at whole and ragged depths of one to nine k-tiles (the sweeps with resident
    samples up to 512, the tile engines beyond), batches that end inside a tile and lists that end inside a chunk."""
    from test_gpu_parity import run_and_compare
    print(f"[depths] step D={D} C={C} B={B}", flush=True)
    W, X = synth.unit_rows(31, synth.TID_W, C, D, bf16=True), synth.unit_rows(31, synth.TID_X, B, D, bf16=True)
    y = synth.labels_uniform(31, B, C)
    G = ((np.arange(C)[:, None] * 7 + 1 + np.arange(K)[None, :] * 13) % C).astype(np.int32)
    X[:5] = synth.bf16_round((0.9 * W[y[:5]] + 0.1 * X[:5]).astype(np.float32))   # a few confident samples
    run_and_compare(ks, orc, W, X, y, G, C, M, scale=30.0, grad_scale=4.0, tag=f"D={D}")


@pytest.mark.parametrize("D", [32, 64, 96, 480])
@pytest.mark.parametrize("scale,grad_scale", [(30.0, 0.0), (30.0, -4.0), (0.0, 4.0), (-20.0, 4.0)])
def test_factors_that_the_sweeps_do_not_take(ks, orc, D, scale, grad_scale):
    """No gradient wanted, ascent, a scale of zero or below: the step as one and as two calls, the loop's call with the next
    batch's selection, the full softmax.  Rows within gradcheck's allowance (the absolute values of the factors are its factors)."""
    import torch
    from gradcheck import check_rows, grad_floors
    print(f"[depths] factors D={D} scale={scale} grad_scale={grad_scale}", flush=True)
    C, B, K, M, alpha = 900, 70, 6, 400, -0.5
    W, X = synth.unit_rows(33, synth.TID_W, C, D, bf16=True), synth.unit_rows(33, synth.TID_X, B, D, bf16=True)
    y, G = synth.labels_uniform(33, B, C), synth.graph_synthetic(33, C, K)
    active, A, tpos = orc.select_active(y, G, C, M)
    Wd, Xd, yd, Gd = dev(W, True), dev(X, True), dev(y), dev(G)

    def check(got, ref, W_A, tp, name):
        floors = [np.abs(f) for f in grad_floors(W_A, X, tp, ref["lse"], scale, grad_scale / B)]
        assert np.abs(got["loss_per_sample"].cpu().numpy() - ref["loss_i"]).max() <= 1e-3 * max(1.0, np.abs(ref["loss_i"]).max())
        check_rows(got["dX"].cpu().numpy(), ref["dX"], floors[0], f"{name} dX")
        check_rows(got["dW"].cpu().numpy()[:W_A.shape[0]], ref["dW"], floors[1], f"{name} dW")

    ref = orc.knn_softmax_fwd_bwd(W, X, active[:A], tpos, scale, grad_scale)
    ref["dW"] = ref["dWA"]
    a = ks.knn_softmax_fwd_bwd(Wd, Xd, yd, Gd, M, scale, grad_scale)
    Wm, Wb = dev(W), Wd.clone()
    b = ks.knn_softmax_fwd_bwd_update(Wm, Wb, Xd, yd, Gd, M, scale, grad_scale, alpha, want_dW=True)
    y2 = dev(synth.labels_uniform(34, B, C))
    Wm2, Wb2 = dev(W), Wd.clone()
    lst = {k: a[k].clone() for k in ("active_idx", "n_active", "target_pos")}
    c, nxt = ks.knn_softmax_fwd_bwd_update_selected_next(Wm2, Wb2, Xd, lst["active_idx"], lst["n_active"], lst["target_pos"], y2, Gd, scale,
                                                         grad_scale, alpha, want_dW=True)
    sel = ks.knn_select_active(y2, Gd, C, M)
    f = ks.full_softmax_fwd_bwd(Wd, Xd, yd, scale, grad_scale)
    torch.cuda.synchronize()
    for out in (a, b, c):
        assert int(out["dev_status"]) == 0
        check(dict(out, dW=out["dW_active"]), ref, W[active[:A]], tpos, "step")
    assert torch.equal(nxt["active_idx"], sel[0]) and torch.equal(nxt["n_active"], sel[1]) and torch.equal(nxt["target_pos"], sel[2])
    assert torch.equal(Wm, Wm2) and torch.equal(Wb, Wb2)
    eW, _ = orc.apply_weight_grad(W, active[:A], b["dW_active"][:A].cpu().numpy(), alpha, want_bf16=False)
    assert np.array_equal(Wm.cpu().numpy(), eW)
    fref = orc.full_softmax_fwd_bwd(W, X, y, scale, grad_scale)
    fref["lse"] = np.log(np.exp(scale * (X.astype(np.float64) @ W.astype(np.float64).T)).sum(axis=1))
    check(f, fref, W, y, "full softmax")


@pytest.mark.parametrize("D", [32, 96, 128])
def test_more_samples_than_the_sweeps_have_workgroups_for(ks, orc, D):
    """65,536 samples and a tile more (256 blocks of 256 samples are the most a sweep takes)."""
    import torch
    from gradcheck import check_rows, grad_floors
    C, B = 300, 65_600
    print(f"[depths] full softmax D={D} B={B}", flush=True)
    W, X = synth.unit_rows(35, synth.TID_W, C, D, bf16=True), synth.unit_rows(35, synth.TID_X, B, D, bf16=True)
    y = synth.labels_uniform(35, B, C)
    f = ks.full_softmax_fwd_bwd(dev(W, True), dev(X, True), dev(y), 20.0, 4.0)
    torch.cuda.synchronize()
    ref = orc.full_softmax_fwd_bwd(W, X, y, 20.0, 4.0)
    lse = np.log(np.exp(20.0 * (X.astype(np.float64) @ W.astype(np.float64).T)).sum(axis=1))
    floors = grad_floors(W, X, y, lse, 20.0, 4.0 / B)
    assert np.abs(f["loss_per_sample"].cpu().numpy() - ref["loss_i"]).max() <= 1e-3 * np.abs(ref["loss_i"]).max()
    check_rows(f["dX"].cpu().numpy(), ref["dX"], floors[0], "dX")
    check_rows(f["dW"].cpu().numpy(), ref["dW"], floors[1], "dW")


@pytest.mark.parametrize("D", [32, 64, 96, 224, 480, 544])
def test_infinite_weights_in_the_last_elements_of_a_row(ks, orc, D):
    """The padding of a ragged depth takes no part.  Graph: a row with an infinite element is the first neighbour of the rows
    whose sign agrees, and takes its own in ascending order of their ids.  Step: a class that every sample's logit is -inf for has
    probability 0, and losses and gradients are those without it (where the infinity itself is not a factor)."""
    import torch
    print(f"[depths] infinite weights D={D}", flush=True)
    C, K, d, c = 200, 8, D - 30, 37
    W = synth.unit_rows(36, synth.TID_W, C, D, bf16=True)
    Wi = W.copy()
    Wi[c, d] = np.inf
    g, s = ks.knn_graph_build(dev(Wi, True), K, want_sims=True)
    torch.cuda.synchronize()
    g, s = g.cpu().numpy(), s.cpu().numpy()
    with np.errstate(invalid="ignore"):
        S = Wi.astype(np.float64) @ Wi.astype(np.float64).T
    others = W[:, d] != 0                                         # (infinity times zero is no similarity)
    for i in np.nonzero(others)[0]:
        S[i, i] = -np.inf
        if i != c or others.all():
            assert np.array_equal(g[i], np.argsort(-S[i], kind="stable")[:K]) and np.isinf(s[i, 0]) == (np.inf in S[i])
    B, M = 40, 190
    X = np.abs(synth.unit_rows(36, synth.TID_X, B, D, bf16=True)) + np.float32(2.0 ** -9)   # every x[d] > 0
    X = synth.bf16_round(X)
    Wi[c, d] = -np.inf
    y = np.array([v for v in synth.labels_uniform(36, 4 * B, C) if v != c][:B], np.int32)
    G = synth.graph_synthetic(36, C, K)
    G[y[0], 0] = c                                                # the class is active
    active, A, tpos = orc.select_active(y, G, C, M)
    assert c in active[:A]
    keep = active[:A][active[:A] != c]
    ref = orc.knn_softmax_fwd_bwd(W, X, keep, np.searchsorted(keep, y).astype(np.int32), 20.0, 2.0)
    out = ks.knn_softmax_fwd_bwd(dev(Wi, True), dev(X, True), dev(y), dev(G), M, 20.0, 2.0)
    torch.cuda.synchronize()
    dX, dW = out["dX"].cpu().numpy(), out["dW_active"][:A].cpu().numpy()[active[:A] != c]
    assert np.abs(out["loss_per_sample"].cpu().numpy() - ref["loss_i"]).max() <= 1e-3 * np.abs(ref["loss_i"]).max()
    for got, want in ((np.delete(dX, d, 1), np.delete(ref["dX"], d, 1)), (dW, ref["dWA"])):
        assert np.linalg.norm(got - want) <= 2e-2 * np.linalg.norm(want)


@pytest.mark.parametrize("D", [32, 64, 96, 192, 320, 384, 480, 576])
def test_unit_rows_flag_has_no_effect_without_a_one_sweep_form(ks, D):
    """The one-sweep softmax rounds X / sum and the own class's gradient once more, which callers at D = 128, 256 and 512 choose
    with the flag; at every other depth losses and gradients are the same bits with and without it."""
    import torch
    print(f"[depths] flag D={D}", flush=True)
    C, B, K, M = 3000, 300, 9, 2500
    W, X = dev(synth.unit_rows(32, synth.TID_W, C, D, bf16=True), True), dev(synth.unit_rows(32, synth.TID_X, B, D, bf16=True), True)
    y, G = dev(synth.labels_uniform(32, B, C)), dev(synth.graph_synthetic(32, C, K))
    a, b = (ks.knn_softmax_fwd_bwd(W, X, y, G, M, 30.0, 4.0, unit_rows=u) for u in (False, True))
    torch.cuda.synchronize()
    n = int(a["n_active"])
    assert int(b["dev_status"]) == 0 and torch.equal(a["loss_per_sample"], b["loss_per_sample"])
    assert torch.equal(a["dX"], b["dX"]) and torch.equal(a["dW_active"][:n], b["dW_active"][:n])
    if D % 64 == 0:   # a node's statistics: normalised to a sum of 1, as without the flag
        s = ks.knn_softmax_fwd_stats(W, X, a["active_idx"], a["n_active"], a["target_pos"], 30.0, unit_rows=True)
        torch.cuda.synchronize()
        assert bool((s["row_sumexp"] == 1.0).all())


@pytest.mark.parametrize("C,D,B,K,M,few", [(60_000, 512, 2048, 32, 49_151, 0), (60_000, 512, 2048, 32, 49_152, 0), (60_001, 512, 1793, 32, 50_011, 0),
                                           (60_000, 512, 2048, 3, 60_000, 50), (60_000, 256, 3841, 16, 50_001, 0), (56_000, 768, 1537, 34, 55_001, 900)])
@pytest.mark.parametrize("unit", [True, False])
def test_feature_gradient_of_large_batches(ks, C, D, B, K, M, few, unit):
    """Tiles of 256 x 256 of the dX contraction and the last size before them; batches that end inside a tile, lists so short
    (labels from `few` classes) that most shares of the active dimension are empty.  Against fp32 products of the same bf16 rows:
    the logit gradient is stored in bf16, 2^-9 of each of its elements, twice that allowed for the exponential and the sums."""
    import torch
    print(f"[depths] dX C={C} D={D} B={B} M={M} few={few} unit={unit}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5)
    W = torch.nn.functional.normalize(torch.randn((C, D), generator=gen, device="cuda")).to(torch.bfloat16)
    X = torch.nn.functional.normalize(torch.randn((B, D), generator=gen, device="cuda")).to(torch.bfloat16)
    y = torch.randint(0, few or C, (B,), generator=gen, device="cuda", dtype=torch.int32)
    G = ((torch.arange(C, device="cuda")[:, None] * 7 + 1 + torch.arange(K, device="cuda")[None, :] * 13) % C).to(torch.int32)
    out = ks.knn_softmax_fwd_bwd(W, X, y, G, M, 30.0, 4.0, unit_rows=unit)
    n = int(out["n_active"])
    Wa, Xf, pos = W[out["active_idx"][:n].long()].float(), X.float(), out["target_pos"].long()
    P = torch.softmax((30.0 * Xf.double() @ Wa.double().T).float(), 1)
    P[torch.arange(B, device="cuda"), pos] -= 1
    f = 30.0 * 4.0 / B
    want, allowed = f * (P @ Wa), f * (P.abs() @ Wa.abs()) * 2.0 ** -8 + 1e-7
    assert (pos >= 0).all() and ((out["dX"] - want).abs() <= allowed).all()


@pytest.mark.parametrize("K,rank", [(16, 8), (32, 10), (64, 12)])
def test_neighbours_that_crowd_in_a_run_of_ids(ks, orc, K, rank):
    """Classes in order of frequency with norms to match: every row's neighbours are the same few hundred, in the first three
    super-blocks, and half of all rows find all of theirs on the stream side of the symmetric sweep.  The sample is an unlucky
    one (450 rows above its rank-th largest; 32 * rank on average).  No row may be left for the exhaustive search."""
    import torch
    C, D, hubs, above = 30_011, 512, 2304, 450
    assert C * D >= 15_000_000                                    # (the symmetric sweep)
    print(f"[depths] hubs C={C} K={K}", flush=True)
    s = np.arange(C // 32, dtype=np.int64)
    sampled = s * 32 + (((s * 2654435761) & 0xFFFFFFFF) >> 16) % 32
    rng = np.random.default_rng(K)
    in_hub = rng.permutation(sampled[sampled < hubs])
    free = rng.permutation(np.setdiff1d(np.arange(hubs), in_hub))
    n_free = above - rank + 1
    order = np.concatenate([rng.permutation(np.concatenate([in_hub[:rank - 1], free[:n_free]])), in_hub[rank - 1:rank],
                            rng.permutation(np.concatenate([in_hub[rank:], free[n_free:]]))])
    norm = np.ones(C)
    norm[order] = np.linspace(12.0, 8.0, hubs)
    u = synth.unit_rows(41, synth.TID_X, 1, D).astype(np.float64)
    W = norm[:, None] * (u + 0.05 * synth.unit_rows(41, synth.TID_W, C, D))
    W = synth.bf16_round(W.astype(np.float32))
    ws = torch.zeros(ks.knn_graph_build_workspace(C, D, K, 0), dtype=torch.uint8, device="cuda")
    g, sims = ks.knn_graph_build(dev(W, True), K, want_sims=True, ws=ws)
    torch.cuda.synchronize()
    assert _exhaustive_rows(ws, C, np.sqrt((W.astype(np.float64) ** 2).sum(1)).max(), 1) == 0
    rows = np.unique(np.concatenate([synth.class_permutation(41, C)[:100], order[:5], [0, hubs - 1, hubs, C - 1]])).astype(np.int32)
    eg, es = orc.graph_bruteforce(W, K, rows)
    assert (g.cpu().numpy()[rows] == eg).all() and (sims.cpu().numpy()[rows] == es.astype(np.float32)).all()


def _exhaustive_rows(ws, norms, largest, maxima):
    """The rows that went to the exhaustive search.  The workspace begins with the row norms, 1,024 maxima of each matrix, the
    largest norm, their number."""
    import torch
    at = (4 * norms + 255) // 256 * 256 + maxima * 4096
    assert abs(float(ws[at:at + 4].view(torch.float32)) - largest) < 1e-3
    return int(ws[at + 256:at + 260].view(torch.int32))


def _sampled_rows_of(C, every):
    """One row of every 16 or 32 searched ones."""
    s = np.arange(C // every, dtype=np.int64)
    return s * every + (((s * 2654435761) & 0xFFFFFFFF) >> 16) % every


def _searched_sample(ws, norms, maxima, Wv):
    """How many searched rows there are to a sampled one in what a call without exhaustive rows has left in its workspace: the
    list of rows for the exhaustive search follows their number, and then come the sampled rows (bf16)."""
    import torch
    at = 2 * ((4 * norms + 255) // 256 * 256) + maxima * 4096 + 512
    for every in (16, 32):
        rows = torch.from_numpy(_sampled_rows_of(Wv.shape[0], every)).cuda()
        n = rows.numel() * Wv.shape[1] * 2
        if n and torch.equal(ws[at:at + n].view(torch.bfloat16).view(rows.numel(), -1), Wv[rows].to(torch.bfloat16)):
            return every
    return 0


@pytest.mark.parametrize("D,K,every,rank,above", [(128, 16, 16, 10, 1100), (320, 16, 32, 8, 1100), (128, 32, 32, 10, 1200), (128, 64, 32, 12, 1350)])
@pytest.mark.parametrize("residues", [(0, 1, 2, 3), (5,), range(8)])
def test_neighbours_of_one_residue_modulo_8(ks, orc, residues, D, K, every, rank, above):
    """The pass of all rows by all blocks: the two lanes that hold a row see the searched rows with bit 2 of their id clear, or
    set.  All rows share their neighbours, which are all one lane's, or fall to both (one residue, half, any), and the sample is an
    unlucky one (`above` rows above its rank-th largest).  No row may be left for the exhaustive search, in the build (one
    part) or in a hop (several, the neighbours in one of them; its sample is one in 32 for every K and the build's own for
    D = 320 and K > 24)."""
    import torch
    C = 60_000
    print(f"[depths] residues {list(residues)} D={D} K={K}", flush=True)
    ids = np.arange(C)
    hubs = ids[np.isin(ids % 8, list(residues))][:2304]
    sampled = _sampled_rows_of(C, every)
    rng = np.random.default_rng(K)
    in_hub, free = rng.permutation(np.intersect1d(hubs, sampled)), rng.permutation(np.setdiff1d(hubs, sampled))
    n_free = above - rank + 1
    assert in_hub.size >= rank and free.size >= n_free
    order = np.concatenate([rng.permutation(np.concatenate([in_hub[:rank - 1], free[:n_free]])), in_hub[rank - 1:rank],
                            rng.permutation(np.concatenate([in_hub[rank:], free[n_free:]]))])
    norm = np.ones(C)
    norm[order] = np.linspace(12.0, 8.0, order.size)
    u = synth.unit_rows(43, synth.TID_X, 1, D).astype(np.float64)
    W = synth.bf16_round((norm[:, None] * (u + 0.05 * synth.unit_rows(43, synth.TID_W, C, D))).astype(np.float32))
    largest = np.sqrt((W.astype(np.float64) ** 2).sum(1)).max()
    Wd = dev(W, True)
    ws = torch.zeros(ks.knn_graph_build_workspace(C, D, K, 0), dtype=torch.uint8, device="cuda")
    assert ws.numel() < 13_000 * C                                # (one part)
    g, sims = ks.knn_graph_build(Wd, K, want_sims=True, ws=ws)
    torch.cuda.synchronize()
    assert _exhaustive_rows(ws, C, largest, 1) == 0
    assert _searched_sample(ws, C, 1, Wd) == every
    rows = np.unique(np.concatenate([synth.class_permutation(43, C)[:60], order[:5], [0, C - 1]])).astype(np.int32)
    eg, es = orc.graph_bruteforce(W, K, rows)
    assert (g.cpu().numpy()[rows] == eg).all() and (sims.cpu().numpy()[rows] == es.astype(np.float32)).all()
    n = 2000
    lists = torch.full((n, K), -1, dtype=torch.int32, device="cuda")
    best = torch.full((n, K), -np.inf, dtype=torch.float64, device="cuda")
    ws = torch.zeros(ks.knn_graph_update_workspace(n, C, D, K, 0), dtype=torch.uint8, device="cuda")
    ks.knn_graph_update(Wd[C - n:].contiguous(), Wd, C - n, 0, lists, best, ws=ws)
    torch.cuda.synchronize()
    assert _exhaustive_rows(ws, n, largest, 2) == 0
    assert _searched_sample(ws, n, 2, Wd) == 32
    assert torch.equal(lists, g[C - n:])


def test_candidate_counts_of_many_rows_fit(ks):
    """Rows of any direction, more than 32 neighbours: the number of candidates is spread widely (a row in 25,000 has 1,024 or
    more), and none may overflow what a row has room for."""
    import torch
    C, D, K = 65_000, 64, 40
    print("[depths] candidate counts", flush=True)
    W = synth.unit_rows(44, synth.TID_W, C, D, bf16=True)
    ws = torch.zeros(ks.knn_graph_build_workspace(C, D, K, 0), dtype=torch.uint8, device="cuda")
    assert ws.numel() < 13_000 * C                                # (one part)
    ks.knn_graph_build(dev(W, True), K, ws=ws)
    torch.cuda.synchronize()
    assert _exhaustive_rows(ws, C, np.sqrt((W.astype(np.float64) ** 2).sum(1)).max(), 1) == 0


@pytest.mark.parametrize("D,A,B", [
    (64, 2, 1), (128, 63, 33), (320, 65, 64), (128, 4097, 65),       # tiles of 64 x 128: two rows, one short, one over, many
    (512, 4737, 40), (320, 5000, 33), (512, 6529, 33), (512, 6527, 129),   # 128 x 128
    (512, 8200, 33), (512, 11_999, 129),                             # 128 x 256
    (2048, 4225, 40), (2048, 6209, 33)])                             # 192 x 256, 256 x 256
def test_gradient_rows_and_update_in_every_tile_shape(ks, orc, D, A, B):
    """The dW launch picks its tile from the active count: lists that end inside a tile of each shape, depths that end inside
    one.  Gradient rows against the oracle, rows beyond the list untouched, the update bit for bit the stand-alone one."""
    _gradient_rows_and_update(ks, orc, D, A, B, False)


@pytest.mark.parametrize("D,A,B", [
    (128, 401, 333), (128, 4097, 333), (256, 6529, 129),             # 64 x 128
    (512, 4737, 333), (128, 20_001, 200), (256, 13_000, 65),         # 128 x 128
    (512, 8200, 333), (256, 18_001, 130),                            # 128 x 256
    (512, 17_425, 333), (128, 33_001, 64), (256, 33_000, 127),       # 192 x 256
    (512, 32_374, 130)])                                             # 256 x 256
def test_target_entries_in_every_tile_shape(ks, orc, D, A, B):
    """Unit rows: the samples' own entries are put into the tiles in LDS, in every shape, over more k-tiles than have their entries
    there at a time, with batches that end inside one and classes that several samples share."""
    _gradient_rows_and_update(ks, orc, D, A, B, True)


def _gradient_rows_and_update(ks, orc, D, A, B, unit):
    import torch
    from gradcheck import check_rows, grad_floors
    print(f"[depths] dW tiles D={D} A={A} B={B} unit={unit}", flush=True)
    C, M, scale, gs, alpha = A + 77, A + 13, 20.0, 4.0, -0.5
    W, X = synth.unit_rows(41, synth.TID_W, C, D, bf16=True), synth.unit_rows(41, synth.TID_X, B, D, bf16=True)
    active = np.sort(synth.class_permutation(41, C)[:A]).astype(np.int32)
    tpos = ((np.arange(B) * 7919 + A - 1) % A).astype(np.int32)
    if unit:
        tpos[B // 2:] = tpos[:B - B // 2]
    act = np.full(M, -1, np.int32)
    act[:A] = active
    Wm, Wb, n = dev(W), dev(W, True), dev(np.array([A], np.int32))
    out = dict(loss_per_sample=torch.empty(B, device="cuda"), loss_mean=torch.empty(1, device="cuda"),
               dX=torch.empty((B, D), device="cuda"), dW_active=torch.full((M, D), 123.0, device="cuda"))
    ks.knn_softmax_fwd_bwd_update_selected(Wm, Wb, dev(X, True), dev(act), n, dev(tpos), scale, gs, alpha, out=out, want_dW=True,
                                           unit_rows=unit)
    Wm2, Wb2 = dev(W), dev(W, True)
    ks.apply_weight_grad(Wm2, Wb2, dev(act), n, out["dW_active"], alpha, idx_sorted_unique=True)
    torch.cuda.synchronize()
    assert int(out["dev_status"]) == 0
    ref = orc.knn_softmax_fwd_bwd(W, X, active, tpos, scale, gs)
    floors = grad_floors(W[active], X, tpos, ref["lse"], scale, gs / B)
    check_rows(out["dX"].cpu().numpy(), ref["dX"], floors[0], "dX")
    check_rows(out["dW_active"][:A].cpu().numpy(), ref["dWA"], floors[1], "dW")
    assert bool((out["dW_active"][A:] == 123.0).all())
    assert torch.equal(Wm, Wm2) and torch.equal(Wb, Wb2) and not torch.equal(Wm, dev(W))


@pytest.mark.parametrize("C,D,B,K,M", [(300, 128, 7, 3, 40), (400, 512, 1, 5, 9), (2000, 256, 8, 6, 70),   # eight samples to a workgroup
                                       (3000, 512, 1000, 1, 1500), (2500, 256, 1024, 1, 1300),             # 32, and fewer shares for dX
                                       (2500, 512, 1030, 1, 1200), (2200, 128, 2001, 0, 2001)])            # 32, shares as they are
def test_one_sweep_combine_beside_the_dx_tiles(ks, orc, C, D, B, K, M):
    """Unit rows: the combine step in workgroups beside the dX tiles, with few and with many samples each, batches that end
    inside a workgroup; confident samples, whose target entries (put into dW's tiles, added to dX) carry the gradient."""
    from test_gpu_parity import run_and_compare
    print(f"[depths] combine D={D} B={B}", flush=True)
    W, X = synth.unit_rows(51, synth.TID_W, C, D, bf16=True), synth.unit_rows(51, synth.TID_X, B, D, bf16=True)
    y = synth.labels_uniform(51, B, C)
    y[B // 2:] = y[: B - B // 2]                                                      # classes with several samples
    G = ((np.arange(C)[:, None] * 7 + 1 + np.arange(K)[None, :] * 13) % C).astype(np.int32)
    X[::3] = synth.bf16_round((0.8 * W[y[::3]] + 0.2 * X[::3]).astype(np.float32))
    run_and_compare(ks, orc, W, X, y, G, C, M, scale=30.0, grad_scale=4.0, tag=f"D={D} B={B}", modes=(True,))


@pytest.mark.parametrize("C,D,K,bf16", [(95, 64, 3, True), (1537, 64, 8, True), (1800, 128, 16, True), (10_000, 128, 8, False), (10_000, 128, 8, True),
                                        (30_001, 64, 32, True), (66_000, 32, 9, True), (58_594, 512, 24, True), (58_593, 512, 24, True),
                                        (46_876, 320, 9, True), (46_875, 320, 9, True), (195_313, 256, 5, True), (195_312, 256, 5, True),
                                        (96_000, 64, 9, True), (96_001, 64, 9, True), (96_001, 128, 8, True), (96_001, 192, 16, True)])
def test_graph_on_both_sides_of_the_denser_sample(ks, orc, C, D, K, bf16):
    """Samples of one row in 16 (less than a chunk, one chunk, several workgroups' lists merged, more blocks than compute units)
    and of one in 32, on either side of the lines between them (C * D = 50, 15 and 30 million, 96,000 rows with K > 8): with
    clustered rows and exact twins.  The sample is the one that was asked for.  No row of bf16 goes to the exhaustive search,
    which finds the right list whatever the thresholds were; of fp32 rows, whose error bound is that of their rounding, at most a few do."""
    import torch
    print(f"[depths] sample C={C} D={D} K={K}", flush=True)
    rng = np.random.default_rng(C)
    centres = synth.unit_rows(61, synth.TID_W, 64, D)
    W = centres[np.arange(C) % 64] + rng.standard_normal((C, D), dtype=np.float32) * (0.7 / np.sqrt(D))
    W /= np.linalg.norm(W, axis=1, keepdims=True)
    W[C - 1] = W[C // 3]
    W = synth.bf16_round(W) if bf16 else W.astype(np.float32)
    rows = np.unique(np.concatenate([rng.integers(0, C, 60), [0, C // 3, C - 1]])).astype(np.int32)
    ws = torch.zeros(ks.knn_graph_build_workspace(C, D, K, 0 if bf16 else 1), dtype=torch.uint8, device="cuda")
    Wd = dev(W, bf16)
    g, s = ks.knn_graph_build(Wd, K, want_sims=True, ws=ws)
    torch.cuda.synchronize()
    eg, es = orc.graph_bruteforce(W, K, rows)
    assert (g.cpu().numpy()[rows] == eg).all() and (s.cpu().numpy()[rows] == es.astype(np.float32)).all()
    if bf16:
        assert _exhaustive_rows(ws, C, float(Wd.double().norm(dim=1).max()), 1) == 0
        most = 50e6 if D <= 256 else 30e6 if D == 512 and K > 16 else 15e6
        symmetric = D in (128, 256, 512) and C * D >= 15e6
        long = not symmetric and K > 8 and (D == 64 or D >= 128) and C > 96_000
        assert _searched_sample(ws, C, 1, Wd) == (16 if K <= 24 and C * D <= most and not long else 32)
    else:
        at = 2 * C * D + (4 * C + 255) // 256 * 256 + 4096 + 256   # (the copy in bf16 comes first)
        assert int(ws[at:at + 4].view(torch.int32)) <= 8


@pytest.mark.parametrize("C_loc,C_vis,D,K", [(40, 7_000, 64, 8), (600, 30_000, 256, 33)])
def test_hop_with_the_sample_in_parts(ks, orc, C_loc, C_vis, D, K):
    """Few local rows against many: the sample's lists come from several workgroups and meet the lists of earlier hops."""
    import torch
    print(f"[depths] hop sample {C_loc} x {C_vis}", flush=True)
    W = synth.unit_rows(62, synth.TID_W, C_loc + 2 * C_vis, D, bf16=True)
    S = W[:C_loc].astype(np.float64) @ W.astype(np.float64).T
    graph = torch.full((C_loc, K), -1, dtype=torch.int32, device="cuda")
    sims = torch.full((C_loc, K), -np.inf, dtype=torch.float64, device="cuda")
    for lo in (C_loc, C_loc + C_vis):
        ks.knn_graph_update(dev(W[:C_loc], True), dev(W[lo:lo + C_vis], True), 0, lo, graph, sims)
    torch.cuda.synchronize()
    best = np.argsort(-S[:, C_loc:], axis=1, kind="stable")[:, :K] + C_loc
    assert (graph.cpu().numpy() == best).all()


@pytest.mark.parametrize("D", [224, 256, 288, 320, 384, 416, 448, 480, 512])
@pytest.mark.parametrize("over", [-1, 1])
def test_two_sweeps_and_one_with_kept_products(ks, orc, D, over):
    """General rows on both sides of the line (512 rows of the batch's tiles times M = 32 D^2) between keeping the first sweep's
    products and sweeping again, at every depth the smaller tests leave to the first."""
    from test_gpu_parity import run_and_compare
    B, K = 300, 63
    M = 32 * D * D // 512 + (over if over > 0 else 0)
    C = M + 400
    print(f"[depths] kept or swept D={D} M={M}", flush=True)
    W, X = synth.unit_rows(71, synth.TID_W, C, D, bf16=True), synth.unit_rows(71, synth.TID_X, B, D, bf16=True)
    W *= 1.25
    y = synth.labels_uniform(71, B, C)
    G = ((np.arange(C)[:, None] * 7 + 1 + np.arange(K)[None, :] * 13) % C).astype(np.int32)
    run_and_compare(ks, orc, W, X, y, G, C, M, scale=20.0, grad_scale=4.0, tag=f"D={D}", modes=(False,))


@pytest.mark.parametrize("D", [32, 64, 96, 128, 192, 256, 320, 384, 448, 480, 512])
@pytest.mark.parametrize("over", [-1, 0, 1])
def test_hop_of_one_to_five_chunks(ks, orc, D, over):
    """Visiting shards of a few rows to a few chunks, whole last chunks and ones of a single row.  (Their parts are too short for
    the halves of a workgroup to take turns: the plain sweep, and for their samples the one in turns with a chunk at most.)  The rows' lists
    are those of all visiting rows."""
    import torch
    K = 8
    for blocks, n in ((0, 10 + over), (0, 32 + over), (1, 96 + over), (1, 128 + over), (2, 256 + over), (3, 384 + over), (5, 640 + over)):
        print(f"[depths] hop of chunks D={D} visiting {n}", flush=True)
        W = synth.unit_rows(61 + blocks, synth.TID_W, n + 70, D, bf16=True)
        Wl, Wv = dev(W[n:], True), dev(W[:n], True)
        graph = torch.full((70, K), -1, dtype=torch.int32, device="cuda")
        sims = torch.full((70, K), -np.inf, dtype=torch.float64, device="cuda")
        ks.knn_graph_update(Wl, Wv, n, 0, graph, sims)
        torch.cuda.synchronize()
        S = W[n:].astype(np.float64) @ W[:n].astype(np.float64).T
        expect = np.argsort(-S, axis=1, kind="stable")[:, :K]
        got = graph.cpu().numpy()
        # (sums in another order: neighbours closer than the rounding of fp64 sums may change places)
        for i in range(70):
            assert (got[i] == expect[i]).all() or np.allclose(S[i, got[i]], S[i, expect[i]], rtol=0, atol=1e-14)


@pytest.mark.parametrize("D", [32, 64, 96, 128, 192, 256, 288, 320, 384, 448, 480, 512])
@pytest.mark.parametrize("last", ["one row", "one chunk", "a chunk and some", "no whole chunks"])
def test_hop_in_turns_with_short_last_parts(ks, orc, D, last):
    """The sweep in turns where the last part has fewer chunks than the pipeline has stages (one of a single row, a whole one, one and
    a piece of the next), and where the parts themselves are no whole number of chunks.  The sizes come from the plan, which says
    that the halves take turns there."""
    import torch
    n_loc, K = 70, 8
    n = size_with_last_part(ks, n_loc, D, K, last)
    if n is None:
        assert last == "no whole chunks" and 96 % ks.knn_graph_recall_plan(n_loc, 20_000, D, K, 0)["chunk"] == 0
        return
    print(f"[depths] hop in turns D={D} visiting {n}: {last}", flush=True)
    gen = torch.Generator().manual_seed(D + n)
    W = torch.nn.functional.normalize(torch.randn((n + n_loc, D), generator=gen)).to(torch.bfloat16)
    W[n:n + 8] = W[n - 8:n]                                       # neighbours among the last part's last rows
    W[n - 1] = W[0]                                               # and a tie: the last row and the first one
    W[n + 8] = W[0]
    graph = torch.full((n_loc, K), -1, dtype=torch.int32, device="cuda")
    sims = torch.full((n_loc, K), -np.inf, dtype=torch.float64, device="cuda")
    ks.knn_graph_update(W[n:].cuda(), W[:n].cuda(), n, 0, graph, sims)
    torch.cuda.synchronize()
    S = (W[n:].double() @ W[:n].double().T).numpy()
    expect = np.argsort(-S, axis=1, kind="stable")[:, :K]
    got = graph.cpu().numpy()
    assert (got[8, :2] == [0, n - 1]).all()
    # (sums in another order: neighbours closer than the rounding of fp64 sums may change places)
    for i in range(n_loc):
        assert (got[i] == expect[i]).all() or np.allclose(S[i, got[i]], S[i, expect[i]], rtol=0, atol=1e-14)


@pytest.mark.parametrize("D", [64, 96, 192, 256, 320, 416, 448, 480])
def test_thresholds_of_many_blocks(ks, orc, D):
    """Enough rows for one workgroup per block in the sample's search (the sweep in turns there too), at depths without the pass that
    computes every similarity once, whole and ragged."""
    import torch
    C, K = 66_000, 12
    print(f"[depths] thresholds D={D}", flush=True)
    W = torch.nn.functional.normalize(torch.randn((C, D), generator=torch.Generator().manual_seed(D))).to(torch.bfloat16)
    g, s = ks.knn_graph_build(W.cuda(), K, want_sims=True)
    torch.cuda.synchronize()
    rows = np.array([0, 1, 255, 256, 31_999, 65_535, 65_536, C - 1], dtype=np.int32)
    eg, es = orc.graph_bruteforce(W.float().numpy(), K, rows)
    assert (g.cpu().numpy()[rows] == eg).all() and (s.cpu().numpy()[rows] == es.astype(np.float32)).all()


@pytest.mark.parametrize("C,K,D,bf16", [(3000, 1, 64, False), (3000, 8, 64, True), (2600, 16, 128, False), (7000, 32, 128, True), (9000, 24, 64, False),
                                        (3000, 40, 64, False), (2600, 29, 320, False), (2600, 32, 320, False),
                                        (118_000, 16, 128, True)])
@pytest.mark.parametrize("noise", [0.0, 0.01, 0.3])
def test_ranking_of_candidates_that_lie_close(ks, orc, C, K, D, bf16, noise):
    """Clusters of 100 rows: more than 64 candidates within the error bound of the K-th (exact copies, and rows closer than the bound of
    rounding fp32 rows), where the search goes through all keys, and rows apart, where it goes through those above the lanes'
    bound; with many segments per row and with three."""
    import torch
    print(f"[depths] close candidates C={C} K={K} D={D} bf16={bf16} noise={noise}", flush=True)
    rng = np.random.default_rng(C + K)
    n = max(C // 100, 1)
    centre = rng.standard_normal((n, D)) / np.sqrt(D)
    W = (centre[np.arange(C) % n] + noise * rng.standard_normal((C, D)) / np.sqrt(D)).astype(np.float32)
    if bf16:
        W = synth.bf16_round(W)
    g, s = ks.knn_graph_build(dev(W, bf16), K, want_sims=True)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([rng.integers(0, C, 40), [0, C - 1]])).astype(np.int32)
    eg, es = orc.graph_bruteforce(W, K, rows)
    assert (g.cpu().numpy()[rows] == eg).all() and (s.cpu().numpy()[rows] == es.astype(np.float32)).all()


@pytest.mark.parametrize("C,K,D,bf16", [(3000, 1, 64, True), (3006, 8, 128, False), (4012, 16, 64, True), (3003, 32, 128, True), (3003, 32, 64, False),
                                        (2000, 30, 160, False), (2013, 32, 320, False)])
@pytest.mark.parametrize("noise", [0.0, 0.05])
def test_ranking_of_exactly_k_close_candidates(ks, orc, C, K, D, bf16, noise):
    """Clusters of K + 1 rows: exactly K candidates above the lanes' bound, all others far below.  (The search among the K ends far below
    the bound then; what the certificate tests against must not.)"""
    import torch
    print(f"[depths] K close candidates C={C} K={K} D={D} bf16={bf16} noise={noise}", flush=True)
    rng = np.random.default_rng(C + K)
    n = C // (K + 1)
    W = rng.standard_normal((n, D))[np.arange(C) % n] + noise * rng.standard_normal((C, D))
    W = (W / np.linalg.norm(W, axis=1, keepdims=True)).astype(np.float32)
    if bf16:
        W = synth.bf16_round(W)
    g, s = ks.knn_graph_build(dev(W, bf16), K, want_sims=True)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([rng.integers(0, C, 200), [0, C - 1]])).astype(np.int32)
    eg, es = orc.graph_bruteforce(W, K, rows)
    assert (g.cpu().numpy()[rows] == eg).all() and (s.cpu().numpy()[rows] == es.astype(np.float32)).all()


@pytest.mark.parametrize("C,D,K,bf16", [(21_484, 512, 32, True), (21_485, 512, 16, True), (21_600, 512, 64, False), (42_968, 256, 24, True), (42_969, 256, 8, True),
                                        (43_008, 256, 33, True)])
def test_graph_around_the_smallest_symmetric_pass(ks, orc, C, D, K, bf16):
    """The last sizes before and the first of the pass that computes every similarity once (C * D = 11 million beyond D = 128)."""
    import torch
    print(f"[depths] symmetric from C={C} D={D} K={K} bf16={bf16}", flush=True)
    assert ks.knn_graph_recall_plan(C, 0, D, K, 0 if bf16 else 1)["kind"] == (2 if C * D >= 11_000_000 else 1)
    W = torch.nn.functional.normalize(torch.randn((C, D), generator=torch.Generator().manual_seed(C))).numpy()
    if bf16:
        W = synth.bf16_round(W)
    W[C - 1] = W[C // 3]                                          # an exact twin
    rows = np.unique(np.concatenate([synth.class_permutation(21, C)[:60], [0, C // 3, C - 2, C - 1]])).astype(np.int32)
    g, s = ks.knn_graph_build(dev(W, bf16), K, want_sims=True)
    torch.cuda.synchronize()
    eg, es = orc.graph_bruteforce(W, K, rows)
    assert (g.cpu().numpy()[rows] == eg).all() and (s.cpu().numpy()[rows] == es.astype(np.float32)).all()
