"""Sampled tensors summed as whole shot counts: a Clifford column side with one to
five quantum outputs (four in registers, more through tiles), with inputs beside
them, with few and many outcomes per variant, at any outcome positions.

The marginal is compared with the contraction of the fragment tensors, formed
separately in fp64 from the same shots: both are sums of at most 4^5 products of
counts below 2^16 times 1/shots, so 1e-12 of the largest entry covers their
rounding, also between the sparse and the dense sum.  A batch agrees with the
calls of its own bit for bit."""
import numpy as np
import pytest

import paper_2303_10788_amd as cc
import workloads as W

pytestmark = pytest.mark.gpu

CLIFF = ["H", "S", "SDG", "X", "Y", "Z", "CX", "CZ"]


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    return cc.Context()


def _circuit(n, outs, ins, seed):
    """`ins` wires prepared by T gates and cut into a Clifford block over n wires, `outs` others cut out of it into
    T gates; the cut-out wires are spread over the block."""
    rng = np.random.default_rng([seed, n, outs, ins])
    wires = [int(w) for w in rng.permutation(n)]
    into, out = wires[:ins], wires[ins:ins + outs]
    ops, cuts = [], []
    for w in into:
        ops += [("H", w, -1, 0.0), ("T", w, -1, 0.0)]
        cuts.append((w, len(ops) - 1))
    ops += W.random_circuit(n, 6 * n, seed, kinds=CLIFF)
    order = [int(w) for w in rng.permutation(n)]
    ops += [("CX", order[i], order[i + 1], 0.0) for i in range(n - 1)]  # one block
    ops += [(("H", "S")[int(rng.integers(2))], w, -1, 0.0) for w in out]
    last = {w: max(i for i, o in enumerate(ops) if w in (o[1], o[2])) for w in out}
    cuts += [(w, last[w]) for w in out]
    for i, w in enumerate(out):
        ops += [("T", w, -1, 0.0), ("H", w, -1, 0.0)]
        if i:
            ops.append(("CX", out[i - 1], w, 0.0))
    return ops, sorted(cuts, key=lambda c: (c[1], c[0]))


def _contract(plan, n_cuts, frags, qubits, shots, seed):
    """2^-k sum_P prod_f T_f[P_f][rows]: the tensors by the fragment call, the sum in numpy."""
    total = np.zeros(1 << len(qubits))
    index = np.arange(1 << len(qubits))
    tensors = []
    for f, (axes, positions) in enumerate(frags):
        T = plan.fragment_tensor(qubits, f, shots=shots, seed=seed)
        row = np.zeros_like(index)
        for bit, p in enumerate(positions):
            row |= ((index >> p) & 1) << bit
        tensors.append((axes, T[:, row]))
    for P in range(4 ** n_cuts):
        term = np.ones(1 << len(qubits))
        for axes, T in tensors:
            term *= T[sum(((P >> (2 * c)) & 3) << (2 * j) for j, c in enumerate(axes))]
        total += term
    return total / 2 ** n_cuts


CASES = [(6, 1, 0, 999), (7, 2, 0, 10000), (9, 3, 0, 65535), (8, 4, 0, 4096), (12, 4, 0, 10000), (11, 5, 0, 777),
         (5, 2, 0, 1), (9, 2, 1, 5000), (9, 1, 2, 3001), (13, 4, 1, 2000), (10, 4, 0, 70000)]


@pytest.mark.parametrize("n,outs,ins,shots", CASES)
def test_marginal_equals_tensor_contraction(ctx, n, outs, ins, shots):
    from oracle import cutting as C
    print(f"counts n={n} outs={outs} ins={ins} shots={shots}", flush=True)
    ops, cuts = _circuit(n, outs, ins, 5)
    plan = cc.Plan(ctx, n, ops, cuts)
    rng = np.random.default_rng(n)
    for qubits in (list(range(n)), sorted(int(q) for q in rng.choice(n, size=n - 2, replace=False))):
        frags = []
        for fr in C.fragment_circuit(n, ops, cuts):
            req = C.make_request(fr, qubits)
            frags.append(([a.cut for a in fr.axes], list(req.req_user)))
        want = _contract(plan, len(cuts), frags, qubits, shots, 3)
        got = plan.marginal(qubits, shots=shots, seed=3)
        assert np.abs(got - want).max() <= 1e-12 * max(1.0, np.abs(want).max())
        sparse = plan.marginal(qubits, shots=shots, seed=3, flags=cc.CCUT_FLAG_SPARSE)
        assert np.abs(sparse - got).max() <= 1e-12 * max(1.0, np.abs(want).max())


def test_batch_equals_calls(ctx):
    print("counts batch", flush=True)
    shots, plans, qubits = 3000, [], []
    for i, (n, outs, ins, _) in enumerate(CASES):
        ops, cuts = _circuit(n, outs, ins, 20 + i)
        plans.append(cc.Plan(ctx, n, ops, cuts))
        qubits.append(list(range(n)))
    got = cc.Batch(ctx, plans, qubits, shots=shots, seed=7).run()
    for i, (p, q) in enumerate(zip(plans, qubits)):
        assert np.array_equal(got[i], p.marginal(q, shots=shots, seed=7, circuit=i)), i


@pytest.mark.parametrize("shots", [20000, 70000])
def test_batch_equals_calls_over_several_shot_blocks(ctx, shots):
    """A variant's shots in more than one block (their counts reduced by a launch over the batch), as 16-bit counts and,
    from 2^16 shots on or as a small plain sum's fold target, as values."""
    print(f"counts batch of {shots} shots", flush=True)
    plans, qubits = [], []
    for i, (n, outs, ins) in enumerate([(6, 1, 0), (7, 2, 0), (8, 4, 0), (9, 2, 1), (9, 1, 2), (8, 1, 1), (7, 0, 2), (6, 0, 3)]):
        ops, cuts = _circuit(n, outs, ins, 40 + i)
        plans.append(cc.Plan(ctx, n, ops, cuts))
        qubits.append(list(range(n)))
    got = cc.Batch(ctx, plans, qubits, shots=shots, seed=7).run()
    for i, (p, q) in enumerate(zip(plans, qubits)):
        assert np.array_equal(got[i], p.marginal(q, shots=shots, seed=7, circuit=i)), i
