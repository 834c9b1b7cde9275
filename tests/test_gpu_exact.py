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


def _blocks(exits, n, depth, seed, n_t=4, tail_near=True):
    """Blocks of 4 wires with the given exit counts, evenly placed, cut one layer before the end where `tail_near` (the
    requested exit wires then keep many columns nonzero)."""
    gap = n // len(exits)
    blocks = [W.Block(list(range(i * gap, i * gap + 4)), list(range(i * gap + 4 - c, i * gap + 4)))
              for i, c in enumerate(exits)]
    ops, cuts = W.block_circuit(n, depth, blocks, t_c=depth - 2 if tail_near else depth // 2, p_cx=0.4, seed=seed, n_t=n_t)
    exits_ = [q for b in blocks for q in b.exits]
    inner = [b.wires[0] for b in blocks]
    return ops, cuts, inner, exits_


@pytest.mark.parametrize("exits,n", [((3, 2), 20), ((3, 3), 40), ((3, 3, 3), 70), ((3, 3, 2, 2), 120)])
def test_columns_fp32_and_learned(ctx, exits, n):
    """Contractions over the nonzero columns (5 to 10 cuts; one and many words of the mask per thread): the fp32 modes
    against fp64, dense and sparse; the term model's norms, support and estimate against the dense tensors' values.  fp32
    bar: the suite's 1e-5; the others as for the dense path (1e-10; norms of exact data exactly)."""
    import torch
    ops, cuts, inner, ex = _blocks(exits, n, 14, n)
    k = len(cuts)
    print(f"columns k={k} n={n}", flush=True)
    plan = cc.Plan(ctx, n, ops, cuts)
    big = max(range(len(exits) + 1), key=lambda f: plan.fragments()[f]["m"])
    for qubits in (sorted(inner + ex[:6]), sorted(inner + ex[:2]), sorted(inner)):
        T = plan.fragment_tensor(qubits, big)
        cols = np.nonzero(np.abs(T).max(axis=1))[0]
        ref = plan.marginal(qubits)
        for flag in (0, cc.CCUT_FLAG_SPARSE):
            for prec in (cc.CCUT_FP32_MFMA_FP64SUM, cc.CCUT_FP32X3_MFMA_FP64SUM):
                got = plan.marginal(qubits, precision=prec, flags=flag)
                assert np.abs(got - ref).max() <= 1e-5
                assert np.array_equal(got, plan.marginal(qubits, precision=prec, flags=flag))
        L = cc.Learned(plan, qubits)
        assert np.abs(L.exhaustive() - ref).max() <= 1e-10
        sup, count = L.support()
        sup = sup.cpu().numpy()
        assert set(sup) <= set(cols) and list(sup) == sorted(sup)
        assert np.abs(cc.Learned(plan, qubits, precision=cc.CCUT_FP32_MFMA_FP64SUM).exhaustive() - ref).max() <= 1e-5
        # a proposal of weights 1..4 over all terms, more on the support: the estimate against the drawn terms' sum
        q = torch.ones(L.K, dtype=torch.float64) / (2 * L.K)
        q[torch.from_numpy(sup.astype(np.int64))] += 0.5 / max(count, 1)
        q = q.cuda()
        terms = torch.empty(700, dtype=torch.int64, device="cuda")
        est = L.estimate(q, 700, seed=3, terms_out=terms)
        w = {}
        frags = plan.fragments()
        tens = {f: plan.fragment_tensor(qubits, f) for f in range(len(frags))}
        exp = np.zeros(1 << len(qubits))
        req = {f: cc.ccut_request_info(plan.handle, qubits, f)[1] for f in tens}
        drawn, times = np.unique(terms.cpu().numpy(), return_counts=True)
        qh = q.cpu().numpy()
        users = {}
        for f, fr in enumerate(frags):
            loc = {wire: i for i, (wire, seg) in enumerate(fr["segments"])}
            last = {}
            for wire, seg in fr["segments"]:
                last[wire] = max(seg, last.get(wire, -1))
            ends = [i for i, (wire, seg) in enumerate(fr["segments"])
                    if seg == sum(1 for c in cuts if c[0] == wire) and wire in qubits]
            users[f] = [qubits.index(fr["segments"][i][0]) for i in ends]
            assert len(users[f]) == req[f]
        idx = np.arange(1 << len(qubits))
        for P, c in zip(drawn, times):
            v = np.full(1 << len(qubits), 0.5 ** k)
            for f, fr in enumerate(frags):
                p = sum(((int(P) >> (2 * a[0])) & 3) << (2 * j) for j, a in enumerate(fr["axes"]))
                b = sum(((idx >> u) & 1) << i for i, u in enumerate(users[f]))
                v = v * tens[f][p][b]
            exp += c * v / (700 * qh[P])
        assert np.abs(est - exp).max() <= 1e-10 * max(1.0, np.abs(exp).max())


@pytest.mark.parametrize("n_in,out,chain,turned", [(13, False, 3, False), (14, False, 3, False), (14, False, 3, True),
                                                   (15, True, 1, False), (15, True, 2, True)])
def test_many_cuts(n_in, out, chain, turned):
    """16 to 18 cuts: n_in one-qubit fragments with a T feed a Clifford part (`out`: one of its wires goes on to a T), and
    `chain` cuts follow one another on a wire of their own; the cuts numbered along the circuit or the other way round."""
    ctx = cc.Context(max_cuts=20)
    rng = np.random.default_rng([n_in, chain])
    n, ops, cuts = n_in + 1, [], []

    def block(q):
        for k in ("H", "T", "H"):
            ops.append((k, q, -1, 0.0))

    for q in range(n_in):
        block(q)
        cuts.append((q, len(ops) - 1))
    for a in range(n_in - 1):
        ops.append(("CX", a, a + 1, 0.0))
    ops.extend(W.random_circuit(n_in, 40, int(rng.integers(1 << 30)), kinds=CLIFF))
    for a in range(n_in - 1):
        ops.append(("CZ", a, a + 1, 0.0))
    if out:
        cuts.append((0, len(ops) - 1 - (n_in - 2)))
        block(0)
    for i in range(chain):
        block(n_in)
        cuts.append((n_in, len(ops) - 1))
    block(n_in)
    if turned:
        cuts = cuts[::-1]
    print(f"many cuts k={len(cuts)}", flush=True)
    plan = cc.Plan(ctx, n, ops, cuts)
    assert plan.info()[0] == n_in + 1 + out + chain + 1
    full = SV.uncut_marginal(n, ops, list(range(n)))
    idx = np.arange(1 << n, dtype=np.uint64)
    masks = np.array([(1 << n) - 1, 1 << n_in | 1, 1 << (n_in - 1), int(rng.integers(1, 1 << n))], dtype=np.uint64)
    par = np.array([[bin(int(x & m)).count("1") & 1 for x in idx] for m in masks])
    assert np.abs(plan.zexpect(masks) - (full * (1 - 2 * par)).sum(axis=1)).max() <= 1e-10
    for qubits in ([0, n_in], [n_in - 1, n_in, 3], [n_in]):
        assert np.abs(plan.marginal(qubits) - SV.uncut_marginal(n, ops, qubits)).max() <= 1e-10
