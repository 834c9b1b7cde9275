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


def test_without_the_native_library(monkeypatch, tmp_path):
    """A missing library, or one that does not load, leaves the conversion to the loop."""
    broken = tmp_path / "broken.so"
    broken.write_bytes(b"not a library")
    for path in (tmp_path / "missing.so", broken):
        monkeypatch.setattr(cc, "PACK_PATH", str(path))
        monkeypatch.setattr(cc, "_PACK", None)
        for ops in GOOD:
            assert bytes(cc._ops_array(ops)) == bytes(_by_op(ops))


def test_the_library_carries_the_interpreter_in_its_name():
    import sysconfig
    from paper_2303_10788_amd import build as B
    assert cc.PACK_PATH == B.PACK_OUT and cc.PACK_PATH.endswith(sysconfig.get_config_var("EXT_SUFFIX"))


def test_a_build_without_the_interpreters_headers(monkeypatch, tmp_path, capfd):
    """It says so, leaves no library of an earlier build behind, and goes on."""
    from paper_2303_10788_amd import build as B
    old = tmp_path / "pack.so"
    old.write_bytes(b"an earlier build")
    monkeypatch.setattr(B, "PACK_OUT", str(old))
    monkeypatch.setattr(B.sysconfig, "get_paths", lambda: {"include": str(tmp_path / "nowhere")})
    B._build_pack()
    assert not old.exists() and list(tmp_path.iterdir()) == []
    assert "Python.h" in capfd.readouterr().err
