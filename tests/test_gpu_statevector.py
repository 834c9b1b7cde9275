"""State-vector kernels at the edges of their shapes: 1 to 12 qubits (fewer
than the three a step acts on, fewer than 16 columns, one and two tiles a
wave), 0 to 6 cut axes of either kind, no, few and all other qubits requested.

Variant tables against the oracle's dense state vector.  Tolerance: every
amplitude is a chain of at most ~150 fused unitaries of 16-term fp64 sums
(relative rounding ~1e-15 each, unitary, so errors add), probabilities at most
1: 1e-12 is far above that and far below any wrong amplitude."""
import numpy as np
import pytest

import paper_2303_10788_amd as cc
import workloads as W
from oracle import cutting as C

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    return cc.Context()


def _fragment(m, n_in, n_out, seed):
    """m wires; n_in of them enter through a cut, n_out of them leave through one; a T on every wire between."""
    rng = np.random.default_rng([m, n_in, n_out, seed])
    wires = rng.permutation(m)
    ops, cuts = [], []
    for q in wires[:n_in]:
        ops.append(("H", int(q), -1, 0.0))
        cuts.append((int(q), len(ops) - 1))
    for q in range(m):
        ops.append(("T", q, -1, 0.0))
    for a, b in zip(range(m - 1), range(1, m)):
        ops.append(("CX", a, b, 0.0))
    ops += W.random_circuit(m, 8 * m, seed, p_two=0.4 if m > 1 else 0.0)
    for q in rng.permutation(m)[:n_out]:
        ops.append(("T", int(q), -1, 0.0))
        cuts.append((int(q), len(ops) - 1))
        ops.append(("H", int(q), -1, 0.0))
    return ops, cuts


@pytest.mark.parametrize("m,n_in,n_out,n_req", [
    (1, 0, 0, 1), (1, 1, 1, 0), (2, 0, 1, 1), (2, 2, 0, 2), (3, 1, 1, 1), (4, 0, 2, 0), (5, 2, 1, 2), (6, 0, 3, 3),
    (6, 3, 0, 6), (7, 1, 2, 2), (8, 0, 0, 8), (8, 4, 0, 8), (8, 0, 4, 4), (9, 2, 2, 5), (9, 3, 2, 1), (10, 0, 2, 0),
    (10, 3, 3, 1), (11, 1, 1, 9), (12, 0, 0, 3), (12, 4, 0, 8), (12, 0, 3, 9), (12, 0, 1, 0)])
def test_variant_tables(ctx, m, n_in, n_out, n_req):
    print(f"state vector m={m} in={n_in} out={n_out} requested={n_req}", flush=True)
    ops, cuts = _fragment(m, n_in, n_out, 5)
    plan = cc.Plan(ctx, m, ops, cuts)
    out_wires = {q for q, a in cuts[n_in:]}
    free = [q for q in range(m) if q not in out_wires]
    rng = np.random.default_rng(m)
    qubits = sorted(int(q) for q in rng.choice(free, size=min(n_req, len(free)), replace=False)) if free else []
    seen = 0
    for f, fr in enumerate(C.fragment_circuit(m, ops, cuts)):
        if fr.clifford:
            continue
        req = C.make_request(fr, qubits)
        got = plan.variant_tables(qubits, f)
        assert got.shape == (fr.n_variants, 1 << len(req.meas))
        step = max(1, fr.n_variants // 48)
        for v in range(0, fr.n_variants, step):
            assert np.abs(got[v] - C.nc_distribution(fr, v, req.meas)).max() <= 1e-12, (f, v)
        assert np.abs(got.sum(axis=1) - 1.0).max() <= 1e-12
        seen = max(seen, fr.m)
    assert seen >= 1


@pytest.mark.parametrize("m,n_out", [(9, 2), (10, 3), (12, 4)])
def test_few_requested_outcomes_take_no_longer(ctx, m, n_out):
    """A fragment's tables when none of its outputs is requested hold a quarter of the entries of those with two requested:
    the state-vector launches take no longer (the least of 20 calls; 1.25 for the events' resolution)."""
    ops, cuts = [], []
    for q in range(m):
        ops += [("H", q, -1, 0.0), ("T", q, -1, 0.0)]
    ops += [("CX", q, q + 1, 0.0) for q in range(m - 1)]
    for q in range(m - n_out, m):
        ops.append(("H", q, -1, 0.0))
        cuts.append((q, len(ops) - 1))
    ops += [("CX", q, m, 0.0) for q in range(m - n_out, m)] + [("CX", m, m + 1, 0.0)]
    plan = cc.Plan(ctx, m + 2, ops, cuts)
    print(f"few outcomes m={m} out={n_out}", flush=True)
    least = []
    for qubits in ([m], [0, 1, m]):
        times = []
        ctx.timing(True)
        for _ in range(20):
            ctx.timing_reset()
            plan.marginal(qubits, method=cc.CCUT_METHOD_VARIANTS)
            times.append(ctx.kernel_times()["sv_kernel"][1])
        ctx.timing(False)
        least.append(min(times))
    assert least[0] <= 1.25 * least[1], least


@pytest.mark.parametrize("m,n_in,n_out,n_req", [(10, 2, 0, 0), (11, 0, 1, 0), (11, 4, 0, 2), (12, 5, 0, 0), (12, 1, 2, 1),
                                                (12, 4, 0, 7)])
def test_variant_tables_of_shared_walks(ctx, m, n_in, n_out, n_req):
    """Two, four and eight waves that share the configurations of the qubits that are not asked for (one where 7 are)."""
    test_variant_tables(ctx, m, n_in, n_out, n_req)
