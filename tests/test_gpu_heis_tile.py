"""Exact tensors of small Clifford fragments in one launch, on one stream with the
state vectors: tiles of 2^11 entries and past them, one requested bit and none, no
and four outputs (and five), 64 qubits and 65, long programs, two such fragments.

Against the uncut state vector or the per-variant path.  Tolerance: products of a
few entries of magnitude <= 4 over at most 4^6 terms scaled by 2^-k: fp64 rounding
below 1e-12; the bar is the suite's 1e-10."""
import numpy as np
import pytest

import paper_2303_10788_amd as cc
import workloads as W
from oracle import statevector as SV
from test_gpu_exact import _circuit

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    return cc.Context()


def _check(ctx, plan, qubits, ref):
    got = [plan.marginal(qubits) for _ in range(4)]  # (later calls replay)
    assert np.abs(got[0] - ref).max() <= 1e-10
    assert np.abs(got[0] - plan.marginal(qubits, method=cc.CCUT_METHOD_VARIANTS)).max() <= 1e-10
    assert all(np.array_equal(g, got[0]) for g in got)
    assert np.array_equal(cc.Batch(ctx, [plan], [qubits]).run()[0], got[0])


@pytest.mark.parametrize("n,n_up,n_down", [(16, 1, 1), (16, 2, 1), (14, 2, 4), (14, 1, 5), (15, 0, 1)])
@pytest.mark.parametrize("clifford_low", [False, True])
def test_tile_edges(ctx, n, n_up, n_down, clifford_low):
    ops, cuts = _circuit(n, n_up, n_down, False, 5)
    if clifford_low:  # the last block Clifford too
        ops = [("S",) + o[1:] if o[0] == "T" and o[1] >= n - 4 - n_down else o for o in ops]
    plan = cc.Plan(ctx, n, ops, cuts)
    mid = [q for q in range(1, n - 4 - n_down)]  # measured wires of the middle fragment
    print(f"tile n={n} up={n_up} down={n_down} mid={len(mid)}", flush=True)
    edge = max(11 - 2 * n_up, 0)  # requested bits that just fit the tile
    for r in sorted({0, 1, min(edge, len(mid)), min(edge + 1, len(mid)), len(mid)}):
        qubits = [n - 1] + mid[:r][::-1] + [0]
        _check(ctx, plan, qubits, SV.uncut_marginal(n, ops, qubits))


@pytest.mark.parametrize("n,depth", [(66, 20), (67, 20), (68, 20), (40, 120), (40, 700)])
def test_words_and_program_lengths(ctx, n, depth):
    ops, cuts = W.block_circuit(n, depth, [W.Block([2, 3, 4, 5], [4, 5])], t_c=depth // 2, p_cx=0.4, seed=n + depth, n_t=2)
    plan = cc.Plan(ctx, n, ops, cuts)
    m = max(f["m"] for f in plan.fragments())
    print(f"n={n} depth={depth} m={m}", flush=True)
    assert n == 40 or 63 <= m <= 67
    qubits = [2, 7, 3] + list(range(9, 15))
    _check(ctx, plan, qubits, plan.marginal(qubits, method=cc.CCUT_METHOD_VARIANTS))
