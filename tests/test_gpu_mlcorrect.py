"""GPU parity of the maximum-likelihood fragment correction (Sec. V-C,
distribution builder) against the oracle (oracle/mlcorrect.py): corrected
variant tables and corrected marginals on sampled Clifford fragments with
one and two quantum outputs and zero to two quantum inputs, the exact-data
fixed point, and the documented refusals.  Bar: 1e-10 (the two sides
diagonalise with different fp64 eigensolvers)."""
import sys

import numpy as np
import pytest

import paper_2303_10788_amd as cc
import workloads as W
from oracle import cutting as C
from oracle import mlcorrect as ML

pytestmark = pytest.mark.gpu

TOL = 1e-10
CLIFF = ("H", "S", "SDG", "X", "Y", "Z", "CX", "CZ")


def _log(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return cc.Context()


def _cases():
    """(name, n, ops, cuts, qubits): every fragment with at most 2 quantum
    outputs, at least one with some."""
    out = []
    w = W.tiny()
    out.append(("tiny", w.n, w.ops, w.cuts, [0, 1, 5]))
    for seed in range(40):
        n = 4 + seed % 5
        ops = W.random_circuit(n, 10 + 4 * n, 300 + seed, kinds=CLIFF)
        k = 1 + seed % 3
        cuts = W.random_cuts(n, ops, k, 300 + seed)
        frags = C.fragment_circuit(n, ops, cuts)
        nout = [sum(a.side == 0 for a in f.axes) for f in frags]
        if max(nout) > 2 or max(nout) == 0:
            continue
        qubits = list(range(0, n, 2)) if seed % 2 else list(range(n))
        out.append((f"clifford{seed}", n, ops, cuts, qubits))
        if len(out) == 9:
            break
    # wider requests: several workgroups of blocks per preparation
    for seed in range(100, 140):
        n = 12
        ops = W.random_circuit(n, 80, 900 + seed, kinds=CLIFF)
        cuts = W.random_cuts(n, ops, 2, 900 + seed)
        nout = [sum(a.side == 0 for a in f.axes) for f in C.fragment_circuit(n, ops, cuts)]
        if 0 < max(nout) <= 2:
            out.append((f"wide{seed}", n, ops, cuts, list(range(n))))
            break
    return out


CASES = _cases()


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("shots", [40, 1000])
def test_corrected_tables_match_oracle(ctx, case, shots):
    name, n, ops, cuts, qubits = CASES[case]
    _log(f"ml tables {name} shots={shots}")
    plan = cc.Plan(ctx, n, ops, cuts)
    frags = C.fragment_circuit(n, ops, cuts)
    for f in frags:
        if not any(a.side == 0 for a in f.axes):
            continue
        req = C.make_request(f, qubits)
        raw = C.variant_distributions(f, req.meas, shots=shots, seed=11)
        want = ML.correct_tables(f, req, raw)
        got = plan.variant_tables(qubits, f.index, shots=shots, seed=11, flags=cc.CCUT_FLAG_ML)
        assert got.shape == want.shape
        assert np.max(np.abs(got - want)) <= TOL, (name, f.index)


@pytest.mark.parametrize("case", range(len(CASES)))
def test_corrected_marginal_matches_oracle(ctx, case):
    name, n, ops, cuts, qubits = CASES[case]
    _log(f"ml marginal {name}")
    plan = cc.Plan(ctx, n, ops, cuts)
    want = C.marginal(n, ops, cuts, qubits, shots=60, seed=5, ml=True)
    got = plan.marginal(qubits, shots=60, seed=5, flags=cc.CCUT_FLAG_ML)
    assert np.max(np.abs(got - want)) <= TOL
    # the correction changed something (sampled data are not physical)
    raw = plan.marginal(qubits, shots=60, seed=5)
    if name != "tiny":
        assert np.max(np.abs(raw - got)) > 1e-6


@pytest.mark.parametrize("case", range(len(CASES)))
def test_exact_tables_are_a_fixed_point(ctx, case):
    name, n, ops, cuts, qubits = CASES[case]
    _log(f"ml fixed point {name}")
    plan = cc.Plan(ctx, n, ops, cuts)
    for f in C.fragment_circuit(n, ops, cuts):
        if not any(a.side == 0 for a in f.axes):
            continue
        raw = plan.variant_tables(qubits, f.index)
        cor = plan.variant_tables(qubits, f.index, flags=cc.CCUT_FLAG_ML)
        assert np.max(np.abs(cor - raw)) <= 1e-12


def test_refusals(ctx):
    # three quantum outputs on one fragment
    ops = [("H", 0, -1, 0.0), ("H", 1, -1, 0.0), ("H", 2, -1, 0.0), ("CX", 0, 1, 0.0), ("CX", 1, 2, 0.0),
           ("S", 0, -1, 0.0), ("S", 1, -1, 0.0), ("S", 2, -1, 0.0)]
    cuts = [(0, 3), (1, 4), (2, 4)]
    plan = cc.Plan(ctx, 3, ops, cuts)
    outs = [sum(a[1] == 0 for a in fr["axes"]) for fr in plan.fragments()]
    assert max(outs) == 3
    with pytest.raises(cc.CcutError) as e:
        plan.marginal([0, 1, 2], shots=100, flags=cc.CCUT_FLAG_ML)
    assert e.value.status == cc.CCUT_E_UNSUPPORTED
    w = W.tiny()
    p2 = cc.Plan(ctx, w.n, w.ops, w.cuts)
    with pytest.raises(cc.CcutError) as e:
        p2.zexpect(np.array([1], dtype=np.uint64), shots=100, flags=cc.CCUT_FLAG_ML)
    assert e.value.status == cc.CCUT_E_UNSUPPORTED


@pytest.mark.parametrize("m,n_out,n_req", [(4, 1, 3), (5, 2, 3), (6, 2, 4), (8, 1, 7), (9, 2, 7), (12, 2, 10)])
def test_state_vector_tables_are_a_fixed_point(ctx, m, n_out, n_req):
    """Physical models whose states have zero eigenvalues (known to rounding): the correction ends and changes nothing."""
    for seed in range(6):
        rng = np.random.default_rng([m, n_out, seed])
        ops = [("H", q, -1, 0.0) for q in range(m)] + [("CX", q, q + 1, 0.0) for q in range(m - 1)]
        ops += W.random_circuit(m, 6 * m, 70 + seed) + [("T", 0, -1, 0.0)]
        outs = sorted(int(q) for q in rng.choice(m, size=n_out, replace=False))
        cuts = []
        for q in outs:
            ops.append(("H", q, -1, 0.0))
            cuts.append((q, len(ops) - 1))
        ops += [("CX", q, m, 0.0) for q in outs]
        qubits = [q for q in range(m) if q not in outs][:n_req]
        _log(f"fixed point m={m} out={n_out} requested={len(qubits)} seed={seed}")
        plan = cc.Plan(ctx, m + 1, ops, cuts)
        for f, fr in enumerate(plan.fragments()):
            if not fr["clifford"]:
                raw = plan.variant_tables(qubits, f)
                cor = plan.variant_tables(qubits, f, flags=cc.CCUT_FLAG_ML)
                assert np.max(np.abs(cor - raw)) <= 1e-12
