"""The state-vector programs' matrices: the gates' product to rounding, whatever
their angles."""
import json

import numpy as np
import pytest

import _hosthip as H

# the step matrices of a plan whose one fragment is not Clifford: 4 bytes by
# 256 and 8 bytes by 256 a step, lane l's A[l % 16][4 c + l / 16], c < 4, of
# the real form of an 8 x 8 unitary
STEPS = """
ops = json.loads({ops!r})
p = cc.Plan(ctx, {n}, [tuple(o) for o in ops], [])
out = np.zeros(1 << {n})
cc.ccut_marginal(p.handle, ctx.handle, cc._eval_opts(), list(range({n})), out)
block = copied()
assert len(p.fragments()) == 1
steps = len(block) // 3072
mats = np.frombuffer(block, dtype=np.float64, offset=1024 * steps).reshape(steps, 64, 4)
result = []
for M in mats:
    A = np.zeros((16, 16))
    for l in range(64):
        for c in range(4):
            A[l % 16, 4 * c + l // 16] = M[l, c]
    result.append([A[:8, :8].tolist(), A[8:, :8].tolist()])
"""


def _steps(n, ops):
    r = H.run(STEPS.format(n=n, ops=json.dumps(ops)))
    return [np.array(re) + 1j * np.array(im) for re, im in r]


S2 = 1 / np.sqrt(2.0)
ONE = {"H": [[S2, S2], [S2, -S2]], "S": [[1, 0], [0, 1j]], "SDG": [[1, 0], [0, -1j]], "X": [[0, 1], [1, 0]],
       "T": [[1, 0], [0, np.exp(0.25j * np.pi)]]}


def _product(ops):
    """The circuit's 8 x 8 unitary, qubit 0 the lowest index bit."""
    U = np.eye(8, dtype=complex)
    for k, a, b, th in ops:
        if k == "CX":
            G = np.zeros((8, 8))
            for i in range(8):
                G[i ^ ((i >> a & 1) << b), i] = 1
        else:
            g = np.array(ONE[k] if k != "RZ" else [[1, 0], [0, np.exp(1j * th)]])
            G = np.zeros((8, 8), dtype=complex)
            for i in range(8):
                for x in (0, 1):
                    G[(i & ~(1 << a)) | (x << a), i] += g[x, i >> a & 1]
        U = G @ U
    return U


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("n,pre,post", [
    (3, [("H", 0, 0, 0.0)], [("CX", 0, 1, 0.0), ("CX", 0, 2, 0.0), ("H", 0, 0, 0.0)]),
    (2, [("H", 0, 0, 0.0), ("CX", 0, 1, 0.0), ("H", 1, 0, 0.0)], [("H", 0, 0, 0.0)]),
    (2, [("H", 0, 0, 0.0), ("T", 0, 0, 0.0), ("CX", 0, 1, 0.0)], []),  # it ends a qubit
    (1, [("H", 0, 0, 0.0)], [])])
def test_an_angle_that_is_no_number_stays(n, pre, post, bad):
    steps = _steps(n, pre + [("RZ", 0, 0, bad)] + post)
    assert any(np.isnan(M).any() for M in steps)


@pytest.mark.parametrize("theta", [1e-14, -1.5e-14, np.pi / 4 + 1e-14, np.pi / 2 - 1.5e-14, np.pi + 2e-14, 1.0])
@pytest.mark.parametrize("pre,post", [(["H"], ["H"]), (["H"], ["SDG", "H"]), (["H", "T"], ["H"])])
def test_an_angle_near_pi_over_four_is_kept(pre, post, theta):
    """The caller's angle, not the multiple of pi / 4 that it lies near.  Tolerance: the products of at most four gates'
    entries of magnitude <= 1 round to within 4 x 2 x 2^-53 < 1e-15; the angles differ by 1e-14 and more, half of it in an
    entry."""
    ops = [(k, 0, 0, 0.0) for k in pre] + [("RZ", 0, 0, theta)] + [(k, 0, 0, 0.0) for k in post]
    (M,) = _steps(1, ops)
    assert np.abs(M - _product(ops)).max() <= 1e-15


def test_clifford_and_t_steps_stay_exact():
    """Matrices of gates without an angle, times sqrt2 where that is so, have the values (a + b / sqrt2) / 64 exactly."""
    ops = [("H", 0, 0, 0.0), ("T", 0, 0, 0.0), ("CX", 0, 1, 0.0), ("H", 1, 0, 0.0), ("T", 1, 0, 0.0), ("H", 0, 0, 0.0),
           ("CX", 1, 2, 0.0), ("T", 2, 0, 0.0), ("H", 2, 0, 0.0)]
    grid = {float(np.float64((a + b * np.longdouble(0.5) ** np.longdouble(0.5)) / 64)) for a in range(-64, 65)
            for b in range(-64, 65)}
    for M in _steps(3, ops):
        assert {float(x) for x in np.concatenate([M.real.ravel(), M.imag.ravel()])} <= grid
