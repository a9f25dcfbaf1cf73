"""One workspace for problems of several sizes: what a caller has sized for its largest batch serves the ragged last one too."""
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


def dev(a, bf16=False):
    import torch
    t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    return t.to(torch.bfloat16) if bf16 else t


def _guarded(nbytes):
    """A workspace of exactly nbytes, and the bytes behind it: all NaN, as bf16 and as fp32."""
    import torch
    whole = torch.full((nbytes + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
    return whole[:nbytes], whole[nbytes:]


def _same(a, b, tag):
    """The same problem with its products kept and swept twice: the slabs' statistics are merged in another order, which moves the
    log-sum-exp by a few units of 2^-24 (|z| <= 20: 1e-5) and an entry of the bf16 gradient by at most one unit of 2^-8."""
    import torch
    torch.cuda.synchronize()
    assert (a["loss_per_sample"] - b["loss_per_sample"]).abs().max() <= 1e-5, tag
    for k in ("dX", "dW_active", "dW"):
        if a.get(k) is not None:
            assert (a[k] - b[k]).norm() <= 2.0 ** -8 * b[k].norm(), (tag, k)


@pytest.mark.parametrize("D,M,large,small", [(512, 14_094, 581, 474), (192, 7_145, 300, 46), (320, 4_074, 774, 500)])
@pytest.mark.parametrize("call", ["step", "selected", "next"])
def test_workspace_of_the_full_batch_serves_the_last_one(ks, call, D, M, large, small):
    """General rows: the smaller batch keeps its products where there is room for them and the larger one does not, so that the
    size query of the smaller one asks for more."""
    import torch
    C, K, scale, gs = M + 500, 8, 20.0, 4.0
    print(f"[workspaces] {call} D={D} M={M} B={large} -> {small}", flush=True)
    size = {"step": lambda B: ks.knn_softmax_workspace(C, D, B, K, M), "selected": lambda B: ks.knn_softmax_selected_workspace(C, D, B, M),
            "next": lambda B: ks.knn_softmax_selected_next_workspace(C, D, B, K, M)}[call]
    if (D, M) == (512, 14_094):
        assert size(large) < size(small)
    W, X = synth.unit_rows(81, synth.TID_W, C, D, bf16=True), synth.unit_rows(81, synth.TID_X, small, D, bf16=True)
    Wb, Xb, y = dev(W, True), dev(X, True), dev(synth.labels_uniform(81, small, C))
    G = dev(((np.arange(C)[:, None] * 7 + 1 + np.arange(K)[None, :] * 13) % C).astype(np.int32))

    def run(ws):
        if call == "step":
            return ks.knn_softmax_fwd_bwd(Wb, Xb, y, G, M, scale, gs, ws=ws)
        act, n, pos, _ = ks.knn_select_active(y, G, C, M)
        if call == "selected":
            return ks.knn_softmax_fwd_bwd_update_selected(None, Wb, Xb, act, n, pos, scale, gs, 0.0, ws=ws)
        nxt = dict(active_idx=torch.empty_like(act), n_active=torch.empty_like(n), target_pos=torch.empty_like(pos))
        out, nxt = ks.knn_softmax_fwd_bwd_update_selected_next(None, Wb, Xb, act, n, pos, y, G, scale, gs, 0.0, next_out=nxt, ws=ws)
        assert torch.equal(nxt["active_idx"], act) and torch.equal(nxt["n_active"], n) and torch.equal(nxt["target_pos"], pos)
        return out

    ws, guard = _guarded(size(large))
    own, own_guard = _guarded(size(small))
    got, want = run(ws), run(own)
    n = int(want["n_active"]) if call == "step" else int(ks.knn_select_active(y, G, C, M)[1])
    for o in (got, want):
        o["dW_active"] = o["dW_active"][:n]
    _same(got, want, call)
    assert bool((guard == 0xFF).all()) and bool((own_guard == 0xFF).all())


def test_workspace_of_all_classes_serves_fewer(ks):
    D, B, large, small, scale, gs = 512, 849, 11_252, 7_600, 20.0, 4.0
    print("[workspaces] full softmax", flush=True)
    assert ks.full_softmax_workspace(large, D, B) < ks.full_softmax_workspace(small, D, B)
    W, X = dev(synth.unit_rows(82, synth.TID_W, small, D, bf16=True), True), dev(synth.unit_rows(82, synth.TID_X, B, D, bf16=True), True)
    y = dev(synth.labels_uniform(82, B, small))
    ws, guard = _guarded(ks.full_softmax_workspace(large, D, B))
    _same(ks.full_softmax_fwd_bwd(W, X, y, scale, gs, ws=ws), ks.full_softmax_fwd_bwd(W, X, y, scale, gs), "full")
    assert bool((guard == 0xFF).all())
