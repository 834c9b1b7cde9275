"""Which calls are captured, replayed and forgotten (the library's host side
over a recording runtime)."""
import pytest

import _hosthip as H

SETUP = """
import workloads as W
w = W.tiny()
p = cc.Plan(ctx, w.n, w.ops, w.cuts)
out = np.zeros(1 << 8)

def call(seed, device, plan=p):
    q = np.array(w.qubits[:2], dtype=np.uint32)
    clear()
    st = cc.lib().ccut_marginal(plan.handle, ctypes.byref(cc._eval_opts(50, seed)), q.ctypes.data_as(cc._U32P), 2,
                                ctypes.c_void_p(out.ctypes.data), device)
    names = [e[0] for e in log()]
    return [st, names.count("begin"), names.count("replay"), names.count("drop")]

"""


def test_host_requests_leave_device_graphs_alone():
    r = H.run(SETUP + """
result = [call(0, 1) for _ in range(3)]
for seed in range(1, 30):
    call(seed, 0)
result += [call(0, 1)]
""")
    eager, capture, replay = [0, 0, 0, 0], [0, 1, 1, 0], [0, 0, 1, 0]
    assert r == [eager, capture, replay, replay]


def test_each_kind_of_call_keeps_eight():
    r = H.run(SETUP + """
for device in (0, 1):
    for seed in range(8):
        for _ in range(7):
            call(seed, device)
result = [call(seed, device)[1:3] for device in (0, 1) for seed in range(8)]
result += [call(8, 0) for _ in range(7)][-1:]          # the ninth: the first one goes
result += [call(0, 0)]
""")
    assert r[:16] == [[0, 1]] * 16
    assert r[16][2] == 1 and r[17][2] == 0


def test_a_host_call_is_captured_late():
    """A capture costs about what five replays save: a host call is captured when it comes a sixth time, a device call the
    second."""
    r = H.run(SETUP + """
result = [[call(3, device) for _ in range(8)] for device in (0, 1)]
""")
    eager, capture, replay = [0, 0, 0, 0], [0, 1, 1, 0], [0, 0, 1, 0]
    assert r == [5 * [eager] + [capture] + 2 * [replay], [eager, capture] + 6 * [replay]]


@pytest.mark.parametrize("device", [0, 1])
@pytest.mark.parametrize("name", ["hipMalloc", "hipHostMalloc"])
def test_a_capture_that_finds_no_memory(name, device):
    """The call runs eagerly instead, and the memory is not asked for again."""
    r = H.run(SETUP + f"""
for seed in range(100, 106):  # the ring of pinned uploads is there
    call(seed, {device})
for _ in range({1 if device else 5}):
    call(7, {device})
fail({name!r})
result = [call(7, {device})]
fail("")
clear()
result += [call(7, {device}), [e[0] for e in log()].count({name!r})]
""")
    assert r == [[0, 0, 0, 0], [0, 0, 0, 0], 0]
