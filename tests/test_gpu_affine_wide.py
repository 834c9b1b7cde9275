"""Sample models of more than 64 measurements at the edges of their words: one
and all 64 measurements in the last word, every number of qubit words, fragments
with more qubits than measurements.  Shot records are compared bit for bit with
literal per-shot stabilizer measurement under the same random words."""
import numpy as np
import pytest

import paper_2303_10788_amd as cc
import workloads as W
from oracle import cutting as C, philox as PX

pytestmark = pytest.mark.gpu

CLIFF = ["H", "S", "SDG", "X", "Y", "Z", "CX", "CZ"]


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    return cc.Context()


@pytest.mark.parametrize("m,measured,gates", [(66, 65, 2), (128, 128, 5), (129, 65, 1), (192, 129, 1), (193, 193, 3),
                                              (256, 250, 1), (321, 256, 1), (385, 65, 2), (449, 400, 1),
                                              (512, 512, 2)])
def test_records_at_word_edges(ctx, m, measured, gates):
    print(f"records m={m} measured={measured}", flush=True)
    chain = [("CX" if q % 3 else "CZ", q, q + 1, 0.0) for q in range(m - 1)]  # one fragment between the cuts
    ops = [("H", 0, -1, 0.0)] + W.random_circuit(m, gates * m, 50 + m, kinds=CLIFF) + chain
    cuts = [(0, 0), (m - 1, len(ops) - 1)]
    ops += W.random_circuit(m - 1, m, 60 + m, kinds=CLIFF)
    rng = np.random.default_rng(m)
    qubits = sorted(int(q) for q in rng.choice(m, size=measured, replace=False))
    plan = cc.Plan(ctx, m, ops, cuts)
    compared = 0
    for f, fr in enumerate(C.fragment_circuit(m, ops, cuts)):
        req = C.make_request(fr, qubits)
        if not fr.clifford or len(req.meas) <= 64:
            continue
        got = plan.shot_records(qubits, f, 0, fr.n_variants, shots=5, seed=41)
        for v in range(fr.n_variants):
            rec = C.clifford_tableau(fr, v).sample(req.meas, 41, PX.variant_id(0, f, v), 0, 5)
            words = np.zeros_like(got[v])
            for j in range(rec.shape[1]):
                words[:, j // 64] |= rec[:, j].astype(np.uint64) << np.uint64(j % 64)
            assert np.array_equal(got[v], words), (f, v)
            compared += 1
    assert compared >= 3


@pytest.mark.parametrize("m,n_ext,shots", [(40, 65, 7), (40, 129, 300), (70, 64, 257), (100, 70, 5), (130, 130, 3)])
def test_parities_at_mask_and_shot_edges(ctx, m, n_ext, shots):
    """Sampled Z strings on both sides of 64 measurements, with mask counts around the groups of 64 and shots that
    fill neither a quad nor a wave, against the oracle: exact parity counts, contraction rounding 1e-12."""
    print(f"parities m={m} masks={n_ext} shots={shots}", flush=True)
    chain = [("CX" if q % 3 else "CZ", q, q + 1, 0.0) for q in range(m - 1)]
    ops = [("H", 0, -1, 0.0)] + W.random_circuit(m, 2 * m, 70 + m, kinds=CLIFF) + chain
    cuts = [(0, 0)]
    rng = np.random.default_rng(m)
    masks = [sum(1 << int(q) for q in rng.choice(m, size=int(rng.integers(1, m + 1)), replace=False))
             for _ in range(n_ext)]
    words = np.array([[(z >> (64 * w)) & 0xFFFFFFFFFFFFFFFF for w in range((m + 63) // 64)] for z in masks],
                     dtype=np.uint64)
    want = C.zexpect(m, ops, cuts, masks, shots=shots, seed=13)
    got = cc.Plan(ctx, m, ops, cuts).zexpect(words, shots=shots, seed=13)
    assert np.abs(got - want).max() <= 1e-12
