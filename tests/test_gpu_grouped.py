"""Several non-Clifford fragments in one call: states of different launch shapes
evolved and combined together, tensors from one launch, with and without a fold
target, and Z strings.  Against the contraction of the fragment tensors, each
formed by its own call (1e-12: fp64 sums of at most 4^5 products of values of
order one), and Z strings against the marginal."""
import numpy as np
import pytest

import paper_2303_10788_amd as cc
import workloads as W
from test_gpu_counts import CLIFF, _contract

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    return cc.Context()


def _circuit(widths, upstream, seed):
    """A Clifford block joined by one wire to a non-Clifford block of each width, which it feeds or (upstream) is fed
    by."""
    rng = np.random.default_rng([seed, *widths])
    ops, cuts, n = [], [], sum(widths)
    first = [sum(widths[:i]) for i in range(len(widths))]

    def block(i):
        w = list(range(first[i], first[i] + widths[i]))
        for q in w:
            ops.append(("H", q, -1, 0.0))
        for _ in range(3):
            for a, b in zip(w, w[1:]):
                ops.append(("CX", a, b, 0.0))
            ops.append(("T", int(rng.choice(w)), -1, 0.0))
            ops.append(("RZ", int(rng.choice(w)), -1, float(rng.normal())))
            ops.append(("H", int(rng.choice(w)), -1, 0.0))

    if upstream:
        for i in range(len(widths)):
            block(i)
            ops.append(("H", first[i], -1, 0.0))
            cuts.append((first[i], len(ops) - 1))
    for a, b in zip(first, first[1:]):
        ops.append(("CX", a, b, 0.0))
    for q in first:
        ops.append((("H", "S", "SDG")[int(rng.integers(3))], q, -1, 0.0))
    for a, b in zip(first, first[1:]):
        ops.append(("CZ", b, a, 0.0))
    if not upstream:
        for i in range(len(widths)):
            cuts.append((first[i], max(k for k, o in enumerate(ops) if first[i] in (o[1], o[2]))))
        for i in range(len(widths)):
            block(i)
    return n, ops, sorted(cuts, key=lambda c: (c[1], c[0]))


@pytest.mark.parametrize("widths", [(1, 1), (2, 3), (1, 8), (7, 8), (2, 9, 3), (4, 11), (1, 2, 3, 4, 5)])
@pytest.mark.parametrize("upstream", [True, False])
def test_marginal_and_strings(ctx, widths, upstream):
    from oracle import cutting as C
    print(f"grouped widths={widths} upstream={upstream}", flush=True)
    n, ops, cuts = _circuit(list(widths), upstream, 3)
    plan = cc.Plan(ctx, n, ops, cuts)
    qubits = list(range(n))
    frags = []
    for fr in C.fragment_circuit(n, ops, cuts):
        frags.append(([a.cut for a in fr.axes], list(C.make_request(fr, qubits).req_user)))
    want = _contract(plan, len(cuts), frags, qubits, 0, 3)
    for method in (cc.CCUT_METHOD_AUTO, cc.CCUT_METHOD_VARIANTS):
        got = plan.marginal(qubits, method=method)
        assert np.abs(got - want).max() <= 1e-12
    rng = np.random.default_rng(n)
    masks = [int(m) for m in rng.integers(1, 1 << n, size=9)]
    index = np.arange(1 << n)
    z = plan.zexpect(np.array([[m] for m in masks], dtype=np.uint64))
    for m, got in zip(masks, z):
        sign = np.array([1 - 2 * (bin(int(i) & m).count("1") & 1) for i in index])
        assert abs(got - (want * sign).sum()) <= 1e-11
