"""State vectors of Clifford gates give whole multiples of 2^-n, to the bit: the
three-qubit steps' matrices are whole multiples of powers of two, with the roots of
two left over taken out of the probabilities.  A T gate on a qubit that stays in
|0> makes the fragment non-Clifford; expected are the oracle's values rounded to
multiples of 2^-n (they are such multiples, known to 1e-14 of at least 2^-12), so
the comparison is for equality."""
import numpy as np
import pytest

import paper_2303_10788_amd as cc
import workloads as W
from oracle import statevector as SV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 4, 7, 9, 12])
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_clifford_states_to_the_bit(n, seed):
    import torch
    assert torch.cuda.is_available()
    ctx = cc.Context()
    rng = np.random.default_rng([n, seed])
    ops = [("T", n - 1, -1, 0.0)]
    for k, a, b, th in W.random_circuit(n - 1, 12 * n + seed, seed, kinds=["H", "S", "SDG", "X", "CX", "CZ"]):
        ops.append((k, a, b, th))
        if rng.random() < 0.2:
            ops.append(("CZ", int(rng.integers(n - 1)), n - 1, 0.0))
    print(f"values n={n} seed={seed} H={sum(o[0] == 'H' for o in ops)}", flush=True)
    plan = cc.Plan(ctx, n, ops, [])
    assert [f["clifford"] for f in plan.fragments()] == [0]
    qubits = list(range(n))
    ref = SV.uncut_marginal(n, ops, qubits)
    want = np.round(ref * 2.0 ** n) / 2.0 ** n
    assert np.abs(want - ref).max() <= 1e-12
    assert np.array_equal(plan.marginal(qubits), want)
    masks = rng.integers(0, 1 << n, size=20).astype(np.uint64)
    par = np.array([[bin(int(x) & int(m)).count("1") & 1 for x in range(1 << n)] for m in masks])
    z = np.array([(want * (1 - 2 * p)).sum() for p in par])
    assert np.array_equal(plan.zexpect(masks), np.round(z))  # -1, 0 or 1


@pytest.mark.parametrize("n", [1, 2, 3, 6, 12])
def test_diagonal_gates_at_the_end(n):
    """T gates that end every qubit change no outcome: the values are those of the Clifford circuit before them, to the
    bit (n = 1: nothing but a T), and the gates still count."""
    import torch
    assert torch.cuda.is_available()
    ctx = cc.Context()
    cliff = list(W.random_circuit(n, 10 * n, n, kinds=["H", "S", "X", "CX", "CZ"])) if n > 1 else []
    ops = cliff + [("T", q, -1, 0.0) for q in range(n)] + [("S", 0, -1, 0.0)]
    print(f"end n={n}", flush=True)
    plan = cc.Plan(ctx, n, ops, [])
    qubits = list(range(n))
    ref = SV.uncut_marginal(n, ops, qubits)
    want = np.round(ref * 2.0 ** n) / 2.0 ** n
    assert np.abs(want - ref).max() <= 1e-12
    assert np.array_equal(plan.marginal(qubits), want)
    one, two = cc.ccut_fragment_ops(plan.handle, 0)
    assert two == sum(o[0] in ("CX", "CZ") for o in ops) and n <= one <= len(ops) - two


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_an_angle_that_is_no_number_shows(bad):
    """Nothing that such a gate reaches is a number: in the circuit's middle every outcome, at a qubit's end those of
    outcome 1 (the matrix there is diag(1, nan))."""
    import torch
    assert torch.cuda.is_available()
    ctx = cc.Context()
    print(f"angle {bad}", flush=True)
    mid = [("H", 0, -1, 0.0), ("RZ", 0, -1, bad)] + [("CX", 0, t, 0.0) for t in (1, 2, 3)] + [("H", 0, -1, 0.0)]
    plan = cc.Plan(ctx, 4, mid, [])
    assert np.isnan(plan.marginal([0, 1, 2, 3])).all() and np.isnan(plan.marginal([2])).all()
    assert np.isnan(plan.zexpect(np.array([1, 2], dtype=np.uint64))).all()
    end = [("H", 0, -1, 0.0), ("T", 0, -1, 0.0), ("CX", 0, 1, 0.0), ("RZ", 1, -1, bad)]
    got = cc.Plan(ctx, 2, end, []).marginal([0, 1])
    assert np.array_equal(np.isnan(got), [False, False, True, True])
