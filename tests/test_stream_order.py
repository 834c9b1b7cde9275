"""What a batch enqueues, in order: a transform starts after every table that it
may read is written, whichever stream wrote it."""
import pytest

import _hosthip as H

BATCH = """
plans, qubits = [], []
for s in range({n}):
    wide = {wide}
    up = [("H", q, 0, 0.0) for q in range(wide)] + [("CX", q, q + 1, 0.0) for q in range(wide)]
    down = [("H", wide, 0, 0.0), ("T", wide, 0, 0.0), ("H", wide, 0, 0.0), ("CX", wide, wide + 1, 0.0)]
    plans.append(cc.Plan(ctx, wide + 2, up + down, [(wide, len(up) - 1)]))
    qubits.append(list(range(wide)) + [wide + 1])
clear()
b = cc.Batch(ctx, plans, qubits, method={method}, use_graph={graph}, shots={shots})
if not {graph}:
    clear()
    b.run()
result = log()
"""


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("n,wide,method,shots", [(2, 2, 1, 0), (5, 2, 1, 0), (11, 3, 1, 0), (3, 15, 0, 0),
                                                 (5, 2, 0, 1000), (5, 2, 0, 70000)])
def test_transforms_follow_their_tables(n, wide, method, shots, graph):
    log = H.run(BATCH.format(n=n, wide=wide, method=method, shots=shots, graph=graph))
    launches = H.launches_before(log)
    writers = ("exact_kernel", "sv_combine", "sample_", "hist_reduce")
    tables = set()
    transforms = 0
    for i, (_, name, _, _, before) in enumerate(launches):
        if "transform_" in name:
            transforms += 1
            assert tables <= before, [launches[t][:3] for t in sorted(tables - before)]
        if any(w in name for w in writers):
            tables.add(i)
    assert transforms and tables


@pytest.mark.parametrize("k,waves", [(1, 1), (2, 1), (3, 8), (4, 8)])
def test_waves_of_a_string_sum(k, waves):
    """A chunk of 64 terms is shared by eight waves; the 4 or 16 terms of one or two cuts are one wave's."""
    log = H.run(f"""
ops, cuts = [], []
for i in range({k} + 1):
    ops += [("H", i, 0, 0.0), ("CX", i, i + 1, 0.0)]
    if i < {k}:
        cuts.append((i + 1, len(ops) - 1))
p = cc.Plan(ctx, {k} + 2, ops, cuts)
clear()
out = np.zeros(5)
cc.ccut_zexpect(p.handle, ctx.handle, cc._eval_opts(100, 1), np.arange(5, dtype=np.uint64)[:, None], out)
result = log()
""")
    (block,) = [b for _, name, _, b, _ in H.launches_before(log) if "zrecombine_small" in name]
    assert block == 64 * waves


@pytest.mark.parametrize("inputs,request_,slices", [(1, 4, 8), (2, 6, 8), (3, 8, 8), (4, 8, 8), (4, 9, 4), (4, 10, 2),
                                                     (5, 9, 1), (6, 10, 1)])
def test_slices_of_a_histogram_reduction(inputs, request_, slices):
    """Few table entries (4^inputs variants of 2^request_) share their shot blocks between up to eight threads each; tables
    that fill the chip by themselves take a thread to an entry."""
    log = H.run(f"""
n = 14
ops, cuts = [], []
for q in range({inputs}):
    ops += [("H", q, 0, 0.0), ("T", q, 0, 0.0), ("H", q, 0, 0.0)]
    cuts.append((q, len(ops) - 1))
for q in range(n - 1):
    ops.append(("CX", q, q + 1, 0.0))
p = cc.Plan(ctx, n, ops, cuts)
clear()
out = np.zeros(1 << {request_})
cc.ccut_marginal(p.handle, ctx.handle, cc._eval_opts(60000, 1), list(range({request_})), out)
result = log()
""")
    (grid,) = [g for _, name, g, _, _ in H.launches_before(log) if "hist_reduce" in name]
    entries = 4 ** inputs << request_
    assert grid == (entries * slices + 255) // 256


@pytest.mark.parametrize("n_in,chain,exact", [(1, 0, True), (1, 2, True), (1, 3, False), (3, 3, False), (4, 2, True),
                                              (4, 3, True)])
def test_strings_through_one_fragment(n_in, chain, exact):
    """Strings take the sum through one Clifford fragment where it is the shorter one: up to two cuts that are not its
    inputs, three from seven cuts on."""
    log = H.run(f"""
n, ops, cuts = {n_in} + 3, [], []
block = lambda q: ops.extend([("H", q, 0, 0.0), ("T", q, 0, 0.0), ("H", q, 0, 0.0)])
for q in range({n_in}):
    block(q)
    cuts.append((q, len(ops) - 1))
for q in range(n - 2):
    ops.append(("CX", q, q + 1, 0.0))
for i in range({chain}):
    block(n - 1)
    cuts.append((n - 1, len(ops) - 1))
block(n - 1)
p = cc.Plan(ctx, n, ops, cuts)
clear()
out = np.zeros(5)
cc.ccut_zexpect(p.handle, ctx.handle, cc._eval_opts(), np.arange(5, dtype=np.uint64)[:, None], out)
result = log()
""")
    names = " ".join(name for _, name, _, _, _ in H.launches_before(log))
    assert ("exact_strings" in names) == exact and ("zrecombine" in names) == (not exact)


@pytest.mark.parametrize("m,inputs,request_,waves", [(9, 0, 0, 1), (10, 2, 0, 2), (11, 4, 3, 4), (12, 4, 0, 8), (12, 5, 6, 8),
                                                     (12, 1, 9, 1), (12, 0, 12, 1)])
def test_waves_of_a_combined_state(m, inputs, request_, waves):
    """The configurations of the qubits that are not asked for which a lane walks through (beyond the six bits of the lanes)
    are shared by up to eight waves, eight or more each."""
    log = H.run(f"""
ops, cuts = [], []
for q in range({inputs}):
    ops += [("H", q, 0, 0.0)]
    cuts.append((q, len(ops) - 1))
for q in range({m}):
    ops += [("H", q, 0, 0.0), ("T", q, 0, 0.0), ("H", q, 0, 0.0)]
for q in range({m} - 1):
    ops.append(("CX", q, q + 1, 0.0))
ops.append(("H", {m}, 0, 0.0))
p = cc.Plan(ctx, {m} + 1, ops, cuts)
clear()
qubits = list(range({request_})) + [{m}]
out = np.zeros(1 << len(qubits))
cc.ccut_marginal(p.handle, ctx.handle, cc._eval_opts(), qubits, out)
result = log()
""")
    (block,) = [b for _, name, _, b, _ in H.launches_before(log) if "sv_combine" in name]
    assert block == 64 * waves
