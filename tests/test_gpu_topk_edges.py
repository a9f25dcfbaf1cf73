"""The last step of a tensor's top-k in its one-pass form: tensors of one chunk at every alignment and around the sizes and
ranks at which the form is left, samples that mislead it, lists of a sampled path around the sizes it holds in registers."""
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


def check(ks, orc, g, offs, k):
    import torch
    print(f"[topk] sizes={np.diff(offs)[:6]} k={k[:6]}", flush=True)
    offs, k = np.asarray(offs, np.int64), np.asarray(k, np.int32)
    idx, val = ks.grad_topk_select(torch.from_numpy(g).cuda(), ks.grad_topk_plan(offs, k))
    torch.cuda.synchronize()
    eidx, eval_ = orc.topk_group(g, offs, k)
    assert np.array_equal(idx.cpu().numpy(), eidx)
    assert np.array_equal(val.cpu().numpy().view(np.uint32), eval_.view(np.uint32))


def grad(seed, n):
    return (synth.normal(seed, synth.TID_GRAD_SET, 0, n) * 1e-2).astype(np.float32)


@pytest.mark.parametrize("n,k", [(2, 1), (7, 3), (9, 8), (63, 1), (64, 16), (65, 17), (257, 100), (1024, 1), (4095, 1000), (4096, 1023),
                                 (4097, 1030), (8191, 512), (8192, 513), (16_000, 511), (16_001, 600), (32_765, 33), (32_767, 512),
                                 (32_768, 513), (32_768, 1), (32_768, 4096)])
def test_tensors_of_one_chunk_at_every_alignment(ks, orc, n, k):
    g = grad(n + k, 4 * n + 6)
    offs = np.cumsum([0, n, 1, n, 1, n, 1, n, 3])                 # element offsets 0, 1, 2, 3 modulo 4 for n = 0 modulo 4, others else
    check(ks, orc, g, offs, [k, 1, k, 1, k, 1, k, 2])


def test_one_chunk_values_that_mislead_the_sample(ks, orc):
    n = 30_000
    a = grad(1, n)
    on, off = a.copy() * 1e-3, a.copy() * 1e-3
    on[::4][:40] = 1.0 + np.arange(40, dtype=np.float32)          # large values on sampled positions only: too few arrive
    off[np.arange(1, n, 4)] = 0.5                                 # a quarter of the tensor equal and unsampled: too many arrive
    runs = np.where(np.arange(n) < 1500, np.float32(2.0), a)      # more equal magnitudes than one bucket ranks
    far = a.copy()
    far[17], far[n - 1], far[5], far[6] = np.inf, -np.float32(3e38), np.nan, -0.0
    g = np.concatenate([on, off, runs, far, np.zeros(n, np.float32), np.full(n, -0.25, np.float32)]).astype(np.float32)
    check(ks, orc, g, np.arange(7) * n, [60, 60, 60, 60, 60, 60])


@pytest.mark.parametrize("n,k", [(32_769, 33), (200_000, 900), (200_000, 1100), (400_000, 3900), (400_000, 4096), (3_000_000, 3000)])
def test_lists_of_the_sampled_path(ks, orc, n, k):
    """Expected list lengths of 4 k: below and above the 4,096 and 16,384 items of the two register forms."""
    g = grad(n + k, n)
    g[: n // 50] *= 40                                            # a heavy tail
    g[n // 2:n // 2 + 3000] = -0.3                                # a run of equal magnitudes
    check(ks, orc, np.concatenate([grad(3, 5), g]), [0, 5, 5 + n], [2, k])


@pytest.mark.parametrize("n,k", [(40_000, 40), (600_000, 600), (2_359_296, 2359), (2_700_000, 2600)])
@pytest.mark.parametrize("kind", ["uniform", "narrow", "normal"])
def test_list_length_of_the_sampled_path_whatever_the_values_are(ks, orc, n, k, kind):
    """The list of a tensor is an order statistic's count, n / 4,096 times a Gamma(r) variable, times at most 3/2 for the
    histogram bin: beyond three times its mean for less than one tensor in a million (r >= 16).  Values that crowd in
    one bin of the first histogram level (uniform ones near their maximum; all of them in [1, 1 + 1 / 64)) are no exception."""
    import torch
    print(f"[topk] list length n={n} k={k} {kind}", flush=True)
    gen = np.random.default_rng(n + k)
    g = {"uniform": lambda: gen.random(n), "narrow": lambda: -1.0 - gen.random(n) / 65.0, "normal": lambda: gen.standard_normal(n)}[kind]().astype(np.float32)
    offs, kk = np.array([0, n], np.int64), np.array([k], np.int32)
    plan = ks.grad_topk_plan(offs, kk)
    ws = torch.zeros(plan.ws_bytes, dtype=torch.uint8, device="cuda")
    idx, val = ks.grad_topk_select(torch.from_numpy(g).cuda(), plan, ws=ws)
    torch.cuda.synchronize()
    nodes = plan.host[32 + 4:].reshape(-1, 12)
    final, thresh = nodes[(nodes[:, 4] & 16) != 0], nodes[(nodes[:, 4] & 4) != 0]
    assert len(final) == len(thresh) == 1
    count, overflow = ws.view(torch.int32)[2 * (int(final[0, 8]) + 1):][:2].tolist()   # the tensor's second workspace word
    r = int(thresh[0, 2])
    print(f"        r={r} count={count} of {r * n / 4096:.0f}", flush=True)
    assert overflow == 0 and k <= count <= 3 * r * n / 4096
    eidx, eval_ = orc.topk_group(g, offs, kk)
    assert np.array_equal(idx.cpu().numpy(), eidx) and np.array_equal(val.cpu().numpy().view(np.uint32), eval_.view(np.uint32))


@pytest.mark.parametrize("sizes,k", [([600_000, 5000, 300_000, 20, 32_768], [600, 10, 4096, 20, 40]),
                                     ([2_400_000, 600_000, 70, 9000], [4096, 500, 7, 9]), ([600_000, 2_400_000], [600, 4096])])
def test_paths_of_every_kind_in_one_group(ks, orc, sizes, k):
    """Sampled paths beside plain trees of three and four levels and tensors of one step."""
    check(ks, orc, grad(7, sum(sizes)), np.cumsum([0] + sizes), k)


def test_plan_saved_before_its_last_level_was_sorted(ks, orc):
    """Plans are plain words that a program may keep in a file.  Those of earlier versions have the last level's steps in tensor
    order (tensors of one step between the last steps of plain trees, whose inputs the level before writes)."""
    import torch
    sizes, k = [600_000, 5000, 300_000, 20, 32_768, 310_000, 9], [600, 10, 4096, 20, 40, 4096, 4]
    offs, k = np.cumsum([0] + sizes).astype(np.int64), np.asarray(k, np.int32)
    host = ks.grad_topk_plan(offs, k).host.copy()
    nodes = host[32 + 4 * len(sizes):].reshape(-1, 12)
    last, n_counted = int(host[6]) - 1, int(host[31])
    assert last == 2 and n_counted == 1
    lo, hi = int(host[8 + 2 * last]) + n_counted, int(host[8 + 2 * last] + host[9 + 2 * last])
    kinds = nodes[lo:hi, 4].tolist()                              # flags: 3 = a tensor of one step, 2 = the last step of a plain tree
    assert kinds == [3, 3, 3, 3, 2, 2] and nodes[lo, 11] == 4
    old = nodes[lo:hi][np.argsort(nodes[lo:hi, 3])]               # by place in the output: tensor order
    old[:, 11] = 0
    nodes[lo:hi] = old
    assert old[:, 4].tolist() == [3, 2, 3, 3, 2, 3]
    g = grad(11, int(offs[-1]))
    idx, val = ks.grad_topk_select(torch.from_numpy(g).cuda(), ks.GradTopkPlan(host, "cuda"))
    torch.cuda.synchronize()
    eidx, eval_ = orc.topk_group(g, offs, k)
    assert np.array_equal(idx.cpu().numpy(), eidx) and np.array_equal(val.cpu().numpy().view(np.uint32), eval_.view(np.uint32))


@pytest.mark.parametrize("n", [4000, 4096, 4200, 20_000, 32_768])
@pytest.mark.parametrize("run", [0.0, -0.375])
def test_one_chunk_with_runs_at_and_around_the_rank(ks, orc, n, run):
    """Most of a tensor zero, or equal: few larger elements, as many as k, one more or fewer; about as many as the one-pass form
    lists; runs of 1,024 elements and a few more above the rest."""
    a = np.sign(grad(n, n)) * (1.0 + np.abs(grad(n, n)))
    at = np.random.default_rng(n).permutation(n)
    g, k = [], []
    for m in (3, 40, 41, 300, 1000, 1024, 1030, 1100, 2000, 3900):
        t = np.full(n, run, np.float32)
        t[at[:m]] = a[at[:m]]
        for kk in sorted({5, 40, min(m, 4096), min(m + 1, 4096)}):
            if kk < n:
                g.append(t)
                k.append(kk)
    for m in (1000, 1024, 1025, 1100):                            # the run is what the ranks fall in
        t = (a * 0.1).astype(np.float32)
        t[at[:m]] = 2.0
        t[at[m:m + 30]] = 3.0
        g += [t, t]
        k += [20, 60]
    check(ks, orc, np.concatenate(g).astype(np.float32), np.arange(len(g) + 1) * n, k)
