"""Exact contractions through one Clifford fragment: no, few and many requested
bits on it (up to several transform passes per workgroup), three to five of
its quantum inputs, cuts that are its outputs or touch it not at all, one and
several words per row.

Against the uncut state vector (up to 16 qubits) or against the per-variant
path of the library (wide circuits).  Tolerance: products of at most four
entries of magnitude <= 2^n_in <= 32 summed over at most 64 terms, the sums
unscaled by 2^(n_in - r - k) <= 1: fp64 rounding below 1e-13; the bar is the
suite's 1e-10."""
import numpy as np
import pytest

import paper_2303_10788_amd as cc
import workloads as W
from oracle import statevector as SV

pytestmark = pytest.mark.gpu
CLIFF = ["H", "S", "SDG", "X", "Z", "CX", "CZ"]


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    return cc.Context()


def _circuit(n, n_up, n_down, side_cut, seed):
    """A block on wires 0..n_up with T gates feeds n_up wires (1..n_up) into a Clifford part on wires 1..n-5; n_down of its
    wires go on into a second block with wires n-4..n-1.  side_cut: a cut inside the second block as well, on wire n-1,
    that touches the Clifford part on neither side."""
    rng = np.random.default_rng([n, n_up, n_down, seed])
    ops, cuts = [], []

    def mix(wires, count, kinds):
        for a, b in zip(wires[:-1], wires[1:]):
            ops.append(("CX", a, b, 0.0))
        for k, a, b, th in W.random_circuit(len(wires), count, int(rng.integers(1 << 30)), kinds=kinds):
            ops.append((k, wires[a], wires[b] if b >= 0 else -1, th))
        for a, b in zip(wires[1:], wires[:-1]):
            ops.append(("CX", a, b, 0.0))

    def last(q):
        return max(i for i, o in enumerate(ops) if q in (o[1], o[2]))

    up = list(range(n_up + 1))
    mix(up, 20, CLIFF + ["T"])
    ops.append(("T", 0, -1, 0.0))
    cuts += [(q, last(q)) for q in up[1:]]
    mid = list(range(1, n - 4))
    mix(mid, 6 * len(mid), CLIFF)
    down = mid[-n_down:] if n_down else []
    cuts += [(q, last(q)) for q in down]
    low = list(range(n - 4, n)) + down
    if side_cut:
        mix([n - 1, n - 2], 6, CLIFF + ["T"])
        cuts.append((n - 1, last(n - 1)))
    mix(low, 20, CLIFF + ["T"])
    ops.append(("T", n - 4, -1, 0.0))
    return ops, cuts


@pytest.mark.parametrize("n,n_up,n_down,side_cut,nq", [
    (14, 3, 0, False, 14), (14, 3, 2, False, 13), (14, 4, 1, True, 12), (16, 3, 3, False, 16), (16, 5, 0, False, 11),
    (15, 4, 2, True, 15)])
def test_against_state_vector(ctx, n, n_up, n_down, side_cut, nq):
    ops, cuts = _circuit(n, n_up, n_down, side_cut, 3)
    print(f"exact n={n} cuts={len(cuts)} nq={nq}", flush=True)
    plan = cc.Plan(ctx, n, ops, cuts)
    assert any(f["clifford"] and sum(a[1] == 1 for a in f["axes"]) >= n_up for f in plan.fragments())
    rng = np.random.default_rng(n)
    for qubits in (sorted(int(q) for q in rng.choice(n, size=nq, replace=False)), [0] + list(range(n - 4, n)) + [2],
                   [int(q) for q in rng.permutation(n)[:nq]]):
        got = plan.marginal(qubits)
        assert np.abs(got - SV.uncut_marginal(n, ops, qubits)).max() <= 1e-10
        assert np.abs(got - plan.marginal(qubits, method=cc.CCUT_METHOD_VARIANTS)).max() <= 1e-10
        assert np.array_equal(cc.Batch(ctx, [plan], [qubits]).run()[0], got)
    masks = rng.integers(0, 1 << n, size=70).astype(np.uint64)
    z = plan.zexpect(masks)
    assert np.abs(z - plan.zexpect(masks, method=cc.CCUT_METHOD_VARIANTS)).max() <= 1e-10
    full = SV.uncut_marginal(n, ops, list(range(n)))
    idx = np.arange(1 << n, dtype=np.uint64)
    for i in (0, 33, 69):
        par = np.array([bin(int(x & masks[i])).count("1") & 1 for x in idx])
        assert abs(z[i] - (full * (1 - 2 * par)).sum()) <= 1e-10


@pytest.mark.parametrize("n,r", [(70, 12), (130, 13), (300, 14)])
def test_wide_against_variants(ctx, n, r):
    """Several words per row, 16 to 64 passes over the subsets; fp32 strings as the plain sum rounds them."""
    ops, cuts = W.block_circuit(n, 16, [W.Block([2, 3, 4, 5, 6], [3, 4, 5, 6])], t_c=6, p_cx=0.35, seed=n, n_t=4)
    print(f"wide n={n} r={r}", flush=True)
    plan = cc.Plan(ctx, n, ops, cuts)
    qubits = [2] + list(range(7, 7 + r))
    assert (256 << len(qubits)) > (1 << 20)  # beyond the plain sum's range
    got = plan.marginal(qubits)
    for flag in (cc.CCUT_FLAG_SPARSE, cc.CCUT_FLAG_SKIP):
        assert np.array_equal(plan.marginal(qubits, flags=flag), got)
    assert np.abs(got - plan.marginal(qubits, method=cc.CCUT_METHOD_VARIANTS)).max() <= 1e-10
    rng = np.random.default_rng(n)
    words = np.zeros((20, (n + 63) // 64), dtype=np.uint64)
    for i in range(20):
        for q in rng.choice(30, size=int(rng.integers(1, 6)), replace=False):
            words[i, 0] |= np.uint64(1 << int(q))
    ref = plan.zexpect(words, method=cc.CCUT_METHOD_VARIANTS)
    assert np.abs(plan.zexpect(words) - ref).max() <= 1e-10
    for prec in (cc.CCUT_FP32_MFMA_FP64SUM, cc.CCUT_FP32X3_MFMA_FP64SUM):
        assert np.abs(plan.zexpect(words, precision=prec) - ref).max() <= 1e-5
