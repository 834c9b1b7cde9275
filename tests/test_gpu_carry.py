"""The Heisenberg carry-back at the edges of its wave layout: one and several
waves of qubits, the last one full or nearly empty, one and several blocks of
64 rows, and a stream too deep for a lane program.

The carried rows decide every sign and random bit of a Clifford fragment, so
shot records (bit for bit against literal per-shot CHP measurement) and exact
Z strings (values -1, 0, 1) show any wrong bit."""
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


@pytest.mark.parametrize("m,n_req", [(2, 1), (63, 40), (64, 62), (65, 9), (128, 61), (129, 60), (192, 62), (257, 20)])
def test_records_over_wave_layouts(ctx, m, n_req):
    print(f"records m={m} requested={n_req}", flush=True)
    ops = [("H", 0, -1, 0.0)] + W.random_circuit(m, 6 * m, 900 + m, kinds=CLIFF)
    last = max(i for i, o in enumerate(ops) if o[1] == m - 1 or o[2] == m - 1)
    cuts = [(0, 0), (m - 1, last)]
    plan = cc.Plan(ctx, m, ops, cuts)
    rng = np.random.default_rng(m)
    qubits = sorted(int(q) for q in rng.choice(m, size=n_req, replace=False))
    seen = 0
    for f, fr in enumerate(C.fragment_circuit(m, ops, cuts)):
        req = C.make_request(fr, qubits)
        if not fr.clifford or not req.meas or len(req.meas) > 64:
            continue
        seen += 1
        got = plan.shot_records(qubits, f, 0, fr.n_variants, shots=11, seed=5)
        for v in range(fr.n_variants):
            exp = C.clifford_tableau(fr, v).sample(req.meas, 5, PX.variant_id(0, f, v), 0, 11).astype(np.uint64)
            words = (exp << np.arange(exp.shape[1], dtype=np.uint64)).sum(axis=1, dtype=np.uint64)
            assert np.array_equal(got[v], words), (m, f, v)
    assert seen


@pytest.mark.parametrize("m", [64, 65, 300, 512])
def test_z_strings_over_row_blocks(ctx, m):
    """130 strings (three blocks of 64 rows) against the uncut stabilizer state's values."""
    print(f"strings m={m}", flush=True)
    ops = W.random_circuit(m, 3 * m, 40 + m, kinds=CLIFF)
    rng = np.random.default_rng(m)
    masks = [sum(1 << int(q) for q in rng.choice(m, size=int(rng.integers(1, 5)), replace=False)) for _ in range(130)]
    words = np.array([[(x >> (64 * w)) & (2 ** 64 - 1) for w in range((m + 63) // 64)] for x in masks], dtype=np.uint64)
    got = cc.Plan(ctx, m, ops, []).zexpect(words)
    exp = C.zexpect(m, ops, [], masks)
    assert np.array_equal(got, exp)


def test_stream_too_deep_for_lanes(ctx):
    """131 000 gates that never leave two wires, on top of a 65-qubit circuit, between two halves of it: six CX in
    turn are the identity, so records and strings equal the shallow circuit's."""
    m = 65
    print("deep stream", flush=True)
    a, b = W.random_circuit(m, 300, 7, kinds=CLIFF), W.random_circuit(m, 300, 8, kinds=CLIFF)
    deep = [("CX", 0, 1, 0.0), ("CX", 1, 0, 0.0)] * 3 * 22_000
    assert len(deep) * 128 > 1 << 24
    rng = np.random.default_rng(3)
    masks = (rng.random((70, m)) < 0.1).astype(np.uint64)
    words = np.zeros((70, 2), dtype=np.uint64)
    for q in range(m):
        words[:, q // 64] |= masks[:, q] << np.uint64(q % 64)
    shallow, long = cc.Plan(ctx, m, a + b, []), cc.Plan(ctx, m, a + deep + b, [])
    assert np.array_equal(long.zexpect(words), shallow.zexpect(words))
    qubits = list(range(3, 60))
    rec = [p.shot_records(qubits, 0, 0, 1, shots=9, seed=2) for p in (long, shallow)]
    assert np.array_equal(rec[0], rec[1])
    outs = [cc.Batch(ctx, [p, p], [[1, 2, 64], [0, 5]], shots=64, seed=3).run() for p in (long, shallow)]
    assert all(np.array_equal(x, y) for x, y in zip(*outs))
