"""The native conversion of a Python circuit equals the op-by-op one, bytes and
errors alike, over what either accepts or refuses."""
import ctypes

import numpy as np
import pytest

import paper_2303_10788_amd as cc
import workloads as W


def _by_op(ops):
    arr = (cc.ccut_op * max(len(ops), 1))()
    for i, (k, a, b, th) in enumerate(ops):
        arr[i] = cc.ccut_op(cc.GATES[k] if isinstance(k, str) else int(k), int(a), int(b) if b >= 0 else 0, 0,
                            float(th))
    return arr


class _Name(str):
    pass


GOOD = [[], W.hwea(20, seed=1).ops, tuple(W.hwea(5, seed=2).ops), [["H", 0, -1, 0.0]], [(6, 1, 2, 0.0)],
        [("RZ", 3, -1, np.float32(0.3))], [("H", -1, -1, 0)], [("CX", 2**31 + 5, 2**32 - 1, 1)],
        [("CX", 2**31 - 1, 2**31 - 1, -1)], [("CX", np.int64(3), np.uint8(4), True)], [("T", 1.9, -0.5, "0.25")],
        [("CZ", 0, -7, 1e-3)], [(_Name("S"), 1, -1, 2**40)], [("RZ", 0, -2**40, -0.0)], [("RZ", True, 0, float("nan"))],
        [("X", 0, -1, 0.0), ("T", 2.0, -1, 0.0)]]
BAD = [[("Q", 0, 0, 0)], [("H", None, 0, 0)], [("H", 0, 0)], [("H", 0, None, 0)], [("H", 0, 0, "x")], [(None, 0, 0, 0)],
       [("H", 0, 0, 10**400)], [([], 0, 0, 0)], [("H", 0, -1, 0.0), 5]]


@pytest.mark.parametrize("i", range(len(GOOD)))
def test_same_rows(i):
    assert bytes(cc._ops_array(GOOD[i])) == bytes(_by_op(GOOD[i]))


@pytest.mark.parametrize("i", range(len(BAD)))
def test_same_errors(i):
    raised = []
    for f in (_by_op, cc._ops_array):
        with pytest.raises(Exception) as e:
            f(BAD[i])
        raised.append((e.type, str(e.value)))
    assert raised[0] == raised[1]


def test_native_path_taken():
    ops = W.hwea(20, seed=1).ops
    arr = (cc.ccut_op * len(ops))()
    pack = cc._pack_lib()
    assert pack(ops, cc.GATES, len(ops), arr) == 0
    assert pack(ops, cc.GATES, len(ops) - 1, arr) == 1
    assert pack(tuple(ops), cc.GATES, len(ops), arr) == 1
