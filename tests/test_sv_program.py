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
