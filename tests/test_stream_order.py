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
