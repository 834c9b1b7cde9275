"""Column norms, shares and phi tables of all fragments of a term model together:
one to 64 and more rows a column, up to 64 partial sums a share, fragments of
unequal sizes, and one without cuts.

Against sums over the fragments' tensors in numpy.  Tolerances: fp32 results of
sums of 2 k logarithms (each at most 40) and of a logarithm of magnitude <= 40:
2 k x 40 x 2^-24 < 1e-4; bf16 features of magnitude <= 1: 2^-9 < 4e-3."""
import numpy as np
import pytest

import paper_2303_10788_amd as cc
from test_gpu_exact import _blocks, _circuit

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    return cc.Context()


def _check(ctx, n, ops, cuts, qubits, **kw):
    k = len(cuts)
    plan = cc.Plan(ctx, n, ops, cuts)
    frags = plan.fragments()
    L = cc.Learned(plan, qubits, **kw)
    K = 4 ** k
    P = np.random.default_rng(k).integers(0, K, size=2000)
    P = np.unique(np.concatenate([P, L.support(cap=K)[0].cpu().numpy()[:2000]]))  # most random terms have no weight
    dig = (P[:, None] >> (2 * np.arange(k))) & 3
    phi = np.full((k, 2, 4), -1.0)
    logw = np.full(len(P), -k * np.log(2.0))  # a term's weight: 2^-k times its norms
    for i, f in enumerate(frags):
        T = plan.fragment_tensor(qubits, i, **kw)
        norm = np.sqrt((T ** 2).sum(axis=1))
        idx = np.zeros(len(P), dtype=np.int64)
        for j, (c, side) in enumerate((a[0], a[1]) for a in f["axes"]):
            d = (np.arange(len(norm)) >> (2 * j)) & 3
            share = np.array([(norm[d == v] ** 2).sum() for v in range(4)]) / (norm ** 2).sum()
            with np.errstate(divide="ignore"):
                phi[c, side] = np.maximum(np.log(share), -40.0) / 40.0
            idx |= dig[:, c] << (2 * j)
        with np.errstate(divide="ignore"):
            logw += np.log(norm[idx])
    import torch
    t = torch.tensor(P, dtype=torch.int64).cuda()
    feats = L.features(t).float().cpu().numpy()[:, :6 * k].reshape(len(P), k, 6)
    want = np.stack([phi[np.arange(k), s, dig] for s in (0, 1)], axis=2)
    assert np.abs(feats[:, :, 4:] - want).max() <= 4e-3
    ys = L.log_weights(t, kind=1).cpu().numpy().astype(np.float64)
    assert np.abs(ys - 40.0 * want.sum(axis=(1, 2))).max() <= 1e-3
    y = L.log_weights(t).cpu().numpy().astype(np.float64)
    live = logw > -25
    assert live.any() and np.abs(y - logw)[live].max() <= 1e-4


@pytest.mark.parametrize("exits,n", [((3, 3), 20), ((3, 3, 2), 26), ((3, 3, 3), 30), ((3, 3, 2, 2), 36)])
def test_many_columns(ctx, exits, n):
    ops, cuts, inner, ex = _blocks(exits, n, 14, n)
    print(f"norms k={len(cuts)} n={n}", flush=True)
    _check(ctx, n, ops, cuts, sorted(inner + ex[:3]))


@pytest.mark.parametrize("n_req", [1, 6, 9, 11])
@pytest.mark.parametrize("shots", [0, 500])
def test_rows_and_a_fragment_without_cuts(ctx, n_req, shots):
    ops, cuts = _circuit(14, 2, 2, False, 7)
    ops = list(ops) + [("H", 14, -1, 0.0), ("T", 14, -1, 0.0), ("H", 14, -1, 0.0)]
    print(f"norms rows n_req={n_req} shots={shots}", flush=True)
    _check(ctx, 15, ops, cuts, ([14] + list(range(1, 8)) + [12, 13, 0])[:n_req], shots=shots, seed=3)
