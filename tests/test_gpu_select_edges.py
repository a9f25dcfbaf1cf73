"""The selection at the edges of its dispatch: the sizes on both sides of the line up to which the selecting workgroups read the
lists themselves, of the line up to which one workgroup's LDS holds a class bitmap, and cuts at every kind of position."""
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


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def check(ks, orc, y, G, C, M):
    import torch
    print(f"[select] C={C} B={len(y)} K={G.shape[1]} M={M}", flush=True)
    a, n, t, st = ks.knn_select_active(dev(y), dev(G), C, M)
    torch.cuda.synchronize()
    ea, eA, et = orc.select_active(y, G, C, M)
    assert int(st.item()) == 0 and int(n.item()) == eA
    assert np.array_equal(a.cpu().numpy(), ea) and np.array_equal(t.cpu().numpy(), et)
    return eA


@pytest.mark.parametrize("C,B,K", [
    (9, 1, 0), (40, 1, 7), (70, 32, 31), (3000, 31, 32), (5000, 64, 31), (5000, 65, 31), (30_000, 128, 63), (30_000, 127, 64),
    (70_000, 512, 15), (70_000, 512, 16), (70_000, 511, 15), (70_000, 513, 14), (1000, 200, 40), (300_000, 16, 120), (255, 100, 50),
    (256, 100, 50), (257, 100, 50), (65_536, 256, 31), (65_537, 256, 31)])
def test_cuts_at_every_kind_of_position(ks, orc, C, B, K):
    """M from the batch size to past what the lists hold, among them exactly the classes seen up to a list position (nothing
    of the next position stays), one more and one fewer, and skewed labels."""
    y = (synth.labels_uniform(4, B, C).astype(np.int64) ** 2 // C).astype(np.int32)
    G = synth.graph_synthetic(4, C, K, locality=4, empty_frac=0.05) if 1 <= K < C else np.full((C, K), -1, np.int32)
    lists = np.concatenate([y[:, None], G[y]], axis=1)
    seen = [len(np.unique(lists[:, :r + 1][lists[:, :r + 1] >= 0])) for r in (0, K // 3, K // 2, max(K - 1, 0), K)]
    floor = max(B, K + 1)
    for M in sorted({m for s in seen for m in (s - 1, s, s + 1) if m >= floor} | {floor, min(C, 2 * floor)}):
        check(ks, orc, y, G, C, M)


@pytest.mark.parametrize("B,over", [(2, 0), (2, 1), (700, 0), (700, 1)])
def test_class_counts_around_the_bitmap_limit(ks, orc, B, over):
    """The largest class count whose bitmap, counts and list fit in LDS, and more (score table)."""
    blocks = (40_600 - 540 - B) // 33                             # of 1,024 classes
    for extra in (0, 1, 1024) if over else (-1023, -1):
        C, K = blocks * 1024 + extra, 12
        c = np.arange(C, dtype=np.int64)[:, None]
        G = ((c + 1 + (c * 2654435761 + np.arange(K) * 40503) % (C - 1)) % C).astype(np.int32)
        y = synth.labels_uniform(9, B, C)
        y[0], y[-1] = C - 1, 0
        check(ks, orc, y, G, C, 13 * B)
        if B > 2:
            check(ks, orc, y, G, C, 5 * B + 3)


def test_batches_larger_than_the_list_in_lds(ks, orc):
    """Many more samples than LDS words, over few and over many classes; the cut bites in the second."""
    for C, B, K, M in [(900, 50_000, 3, 50_000), (60_000, 42_000, 2, 42_000), (60_000, 42_000, 2, 55_000)]:
        y = synth.labels_uniform(5, B, C)
        check(ks, orc, y, synth.graph_synthetic(5, C, K, locality=8, empty_frac=0.0), C, M)


@pytest.mark.parametrize("C,B,K,M", [(3000, 64, 31, 2048), (70_000, 512, 15, 600), (70_000, 300, 0, 300)])
@pytest.mark.parametrize("where", ["target_pos", "active_idx"])
def test_outputs_in_place_of_the_labels(ks, orc, where, C, B, K, M):
    """Positions or list written over the labels, beside work on another stream that makes some workgroups start late."""
    import torch
    G = synth.graph_synthetic(6, C, K, locality=4, empty_frac=0.05) if K else np.full((C, 0), -1, np.int32)
    g = dev(G) if K else None
    W = torch.nn.functional.normalize(torch.randn(40_000, 128, device="cuda"), dim=1).bfloat16()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for seed in range(4):
        y = synth.labels_uniform(20 + seed, B, C)
        print(f"[select in place] {where} C={C} B={B} K={K} seed={seed}", flush=True)
        ea, eA, et = orc.select_active(y, G, C, M)
        shared = torch.full((max(B, M),), -7, dtype=torch.int32, device="cuda")
        labels = shared[:B]
        labels.copy_(dev(y))
        a = shared[:M] if where == "active_idx" else torch.empty(M, dtype=torch.int32, device="cuda")
        t = labels if where == "target_pos" else torch.empty(B, dtype=torch.int32, device="cuda")
        n = torch.empty(1, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            ks.knn_graph_build(W, 8)
        _, _, _, st = ks.knn_select_active_static(labels, g, C, M, out=(a, n, t))
        torch.cuda.synchronize()
        assert int(st.item()) == 0 and int(n.item()) == eA
        assert np.array_equal(a.cpu().numpy(), ea) and np.array_equal(t.cpu().numpy(), et)


@pytest.mark.parametrize("C,B,K", [(30_000, 60, 100), (30_000, 301, 100), (60_000, 512, 127), (500_000, 700, 100)])
@pytest.mark.parametrize("shape", ["late", "early", "steps", "empty"])
def test_counts_that_do_not_grow_evenly(ks, orc, shape, C, B, K):
    """The search of the cut guesses from how many classes the positions bring: all of them at the last ones, at the first ones,
    in runs between runs that bring none (the same classes in every list, or empty entries)."""
    rng = np.random.default_rng(K + B)
    G = rng.integers(0, C, (C, K)).astype(np.int32)
    same = np.broadcast_to(np.arange(K, dtype=np.int32), (C, K))
    quiet = {"late": np.arange(K) < K - 12, "early": np.arange(K) >= 12, "steps": (np.arange(K) // 11) % 2 == 0,
             "empty": (np.arange(K) // 9) % 3 != 2}[shape]
    G[:, quiet] = -1 if shape == "empty" else same[:, quiet]
    y = synth.labels_uniform(8, B, C)
    lists = np.concatenate([y[:, None], G[y]], axis=1)
    seen = [len(np.unique(lists[:, :r + 1][lists[:, :r + 1] >= 0])) for r in range(K + 1)]
    floor = max(B, K + 1)
    for M in sorted({max(floor, m) for s in (seen[5], seen[K // 2], seen[K - 6], seen[K - 1], seen[K]) for m in (s - 1, s, s + 3)} | {floor}):
        check(ks, orc, y, G, C, M)


@pytest.mark.parametrize("B,K,M", [(1000, 99, 60_000), (1001, 99, 60_000), (2000, 99, 174_999), (2000, 99, 175_000), (2000, 99, 120_000),
                                   (4096, 23, 50_000), (4097, 23, 50_000)])
def test_many_classes_and_many_candidates(ks, orc, B, K, M):
    """Both sides of the lines between the bitmap and the score table beyond 393,216 classes."""
    C = 450_000
    check(ks, orc, synth.labels_uniform(10, B, C), synth.graph_synthetic(10, C, K, locality=8, empty_frac=0.0), C, M)
