"""Planning takes time in proportion to the gates."""
import ctypes
import time

import numpy as np
import pytest

import paper_2303_10788_amd as cc


def _seconds(ctx, n, ops):
    """Of creating a plan without cuts (the best of three)."""
    arr, none, best = cc._ops_array(ops), cc._cuts_array([]), float("inf")
    for _ in range(3):
        h = ctypes.c_void_p()
        t = time.perf_counter()
        assert cc.lib().ccut_plan_create(ctx.handle, n, arr, len(ops), none, 0, ctypes.byref(h)) == 0
        best = min(best, time.perf_counter() - t)
        cc.lib().ccut_plan_destroy(h)
    return best


def _circuit(n, busy, gates):
    """All n qubits tied by CX gates, then gates on the busy ones alone."""
    rng = np.random.default_rng([n, busy])
    ops = [("CX", 0, q, 0.0) for q in range(1, n)]
    for two, kind, a, b in zip(rng.random(gates) < 0.4, rng.choice(["H", "S", "T"], gates),
                               rng.integers(0, busy, gates), rng.integers(1, busy, gates)):
        a, b = int(a), int(b)
        ops.append(("CX", a, (a + b) % busy, 0.0) if two else (str(kind), a, -1, 0.0))
    return ops


@pytest.mark.parametrize("n,busy", [(12, 12), (12, 6), (12, 4), (12, 2)])
def test_a_state_vector_fragment(n, busy):
    """16 times the gates take about 16 times as long, not 256 times: at most 64."""
    ctx = cc.Context(device=-1)
    few, many = _seconds(ctx, n, _circuit(n, busy, 2000)), _seconds(ctx, n, _circuit(n, busy, 32000))
    assert many <= 64 * few, (few, many)
