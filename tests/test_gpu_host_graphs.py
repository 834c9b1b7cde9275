"""Host-output calls repeated with the same arguments replay a captured graph from
the second on.  Every result equals the eager one bit for bit, into any buffer, with
larger eager calls (which grow the context's scratch), device-output replays and
other requests in between; more keys than a plan keeps graphs still give their own
results."""
import numpy as np
import pytest

import paper_2303_10788_amd as cc
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    import torch
    assert torch.cuda.is_available()
    return cc.Context()


def _eager(ctx, fn):
    ctx.call_graphs(False)
    try:
        return fn()
    finally:
        ctx.call_graphs(True)


@pytest.mark.parametrize("shots,precision", [(0, cc.CCUT_FP64), (700, cc.CCUT_FP64), (0, cc.CCUT_FP32_MFMA_FP64SUM)])
def test_replays_equal_eager(ctx, shots, precision):
    import torch
    print(f"host graphs shots={shots} precision={precision}", flush=True)
    small, big = W.tiny(), W.mid(shots=shots)
    p, q = cc.Plan(ctx, small.n, small.ops, small.cuts), cc.Plan(ctx, big.n, big.ops, big.cuts)
    opts = dict(shots=shots, seed=3, precision=precision)
    masks = small.zmask_words()
    ref_m = _eager(ctx, lambda: p.marginal(small.qubits, **opts))
    ref_z = _eager(ctx, lambda: p.zexpect(masks, **opts))
    dev = torch.empty(ref_m.size, dtype=torch.float64, device="cuda")
    for rep in range(6):
        out = np.full(ref_m.size, np.nan)  # a buffer of its own each time
        assert np.array_equal(p.marginal(small.qubits, out=out, **opts), ref_m), rep
        assert np.array_equal(p.zexpect(masks, **opts), ref_z), rep
        p.marginal(small.qubits, out=dev, **opts)
        if rep == 2:  # grows the scratch the graphs were captured in
            q.marginal(big.qubits, **opts)
        if rep == 3:  # another request, then the first again
            p.marginal(small.qubits[:2], **opts)
        torch.cuda.synchronize()
        assert np.array_equal(dev.cpu().numpy(), ref_m), rep


def test_more_keys_than_graphs(ctx):
    w = W.tiny()
    plan = cc.Plan(ctx, w.n, w.ops, w.cuts)
    print("host graphs, eleven keys", flush=True)
    refs = [_eager(ctx, lambda s=s: plan.marginal(w.qubits, shots=50, seed=s)) for s in range(11)]
    for rep in range(4):
        for s in range(11):
            for _ in range(1 + rep):
                assert np.array_equal(plan.marginal(w.qubits, shots=50, seed=s), refs[s]), (rep, s)


def test_errors_stay(ctx):
    w = W.tiny()
    plan = cc.Plan(ctx, w.n, w.ops, w.cuts)
    print("host graphs, refused requests", flush=True)
    for _ in range(3):
        with pytest.raises(cc.CcutError):
            plan.marginal([0, 0])
        with pytest.raises(cc.CcutError):
            plan.marginal(w.qubits, flags=cc.CCUT_FLAG_SETTLE)


@pytest.mark.parametrize("shots", [0, 700])
def test_many_repeats(ctx, shots):
    """Twelve equal calls of each kind (eager, captured, replayed), other requests and device calls between them."""
    import torch
    print(f"host graphs, twelve repeats, shots={shots}", flush=True)
    w, other = W.mid(shots=shots), W.tiny()
    p, q = cc.Plan(ctx, w.n, w.ops, w.cuts), cc.Plan(ctx, other.n, other.ops, other.cuts)
    masks = w.zmask_words()
    ref_m = _eager(ctx, lambda: p.marginal(w.qubits, shots=shots, seed=3))
    ref_z = _eager(ctx, lambda: p.zexpect(masks, shots=shots, seed=3))
    dev = torch.empty(ref_m.size, dtype=torch.float64, device="cuda")
    for rep in range(12):
        assert np.array_equal(p.marginal(w.qubits, shots=shots, seed=3), ref_m), rep
        assert np.array_equal(p.zexpect(masks, shots=shots, seed=3), ref_z), rep
        q.marginal(other.qubits, shots=shots, seed=rep)
        p.marginal(w.qubits, shots=shots, seed=3, out=dev)
        torch.cuda.synchronize()
        assert np.array_equal(dev.cpu().numpy(), ref_m), rep
