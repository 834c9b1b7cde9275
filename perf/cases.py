"""Timed cases of the framework: what a user's program has it do, each through the public Python entry points.

A case is a dict of plain values.  The kinds, and what each stands for in use:

* ``marginal``  one circuit's output marginal, asked again with a plan that the program keeps: exact or sampled,
  host or device output, every precision and Clifford flag, 1 to 4 blocks of non-Clifford gates
* ``zexpect``   the same circuit's Z strings (an ansatz's observables): exact or sampled; beyond 64 measured qubits
  the sample models span several words
* ``both``      one marginal and its Z strings per step, as the 400-qubit ladder workload asks them
* ``batch``     many circuits of mixed width, depth and cuts evaluated together (one batch kept, replayed)
* ``scan``      a circuit seen once: cuts found, planned, evaluated exactly and dropped again
* ``learned``   the importance-sampled marginal with the term network as its proposal
* ``train``     a stretch of training of that network, from given parameters to updated ones

Sizes are those of ``workloads``, the tests and the benchmark (8 to 400 qubits, 1 to 10 cuts, 0 to 1e5 shots, 1 to 256
circuits a batch), with odd ones between.
"""
import math

import numpy as np
import torch

import paper_2303_10788_amd as cc
import workloads as W

PRECISION = {"fp64": cc.CCUT_FP64, "fp32": cc.CCUT_FP32_MFMA_FP64SUM, "fp32x3": cc.CCUT_FP32X3_MFMA_FP64SUM}
FLAGS = {"": 0, "sparse": cc.CCUT_FLAG_SPARSE, "skip": cc.CCUT_FLAG_SKIP, "ml": cc.CCUT_FLAG_ML,
         "settle": cc.CCUT_FLAG_SETTLE}


def _one(kind, n, depth, width, exits, n_t, *, shots=0, nq=0, strings=0, weight=0, mirrored=False, topology="random",
         p_cx=0.3, precision="fp64", flag="", out="device"):
    """A case on one circuit; exits: cut wires per block, as text ("3,3,2,2": four blocks); weight: qubits of a Z
    string at most (0: each with probability 1/2)."""
    return dict(kind=kind, n=n, depth=depth, width=width, exits=exits, n_t=n_t, shots=shots, nq=nq, strings=strings,
                weight=weight, mirrored=mirrored, topology=topology, p_cx=p_cx, precision=precision, flag=flag, out=out)


def listed():
    return [
        # the smallest call: one cut, exact, the whole distribution into a host array (latency and launches)
        dict(name="exact_8q_host", **_one("marginal", 8, 10, 4, "1", 2, nq=8, out="host")),
        # an ordinary exact call at odd sizes: Clifford part upstream of a 7-qubit block with three cuts
        dict(name="exact_17q_mirrored", **_one("marginal", 17, 23, 7, "3", 5, nq=15, mirrored=True)),
        # the 32-qubit sampled workload: its 12-qubit marginal, and its 64 random Z strings
        dict(name="sampled_32q_marginal", **_one("marginal", 32, 40, 10, "2", 4, shots=100_000, nq=12)),
        dict(name="sampled_32q_zstrings", **_one("zexpect", 32, 40, 10, "2", 4, shots=100_000, strings=64)),
        # more than 64 measured qubits: an odd number of strings over 161 qubits, read on the host
        dict(name="sampled_161q_zstrings_host", **_one("zexpect", 161, 37, 8, "3", 5, shots=10_000, strings=49,
                                                       out="host")),
        # a small batch of short sampling runs, results read on the host
        dict(name="batch_13x999", kind="batch", circuits=13, shots=999, out="host"),
        # the benchmark's batch: 256 circuits, 1e4 shots a variant, outputs left on the device
        dict(name="batch_256x10000", kind="batch", circuits=256, shots=10_000, out="device"),
        # the 400-qubit ladder: six cuts, exact Clifford tensors, fp32 matrix products, marginal and 64 strings
        dict(name="ladder_400q_fp32", **_one("both", 400, 30, 6, "3,3", 8, nq=16, strings=64, topology="nn", p_cx=0.5,
                                             precision="fp32")),
        # the largest exhaustive sum: ten cuts, 4^10 terms, in fp64
        dict(name="tencuts_300q_exact", **_one("marginal", 300, 50, 5, "3,3,2,2", 12, nq=16)),
        # the same circuit family through the learned proposal, with its standard error
        dict(name="learned_10cuts", **_one("learned", 300, 50, 5, "3,3,2,2", 12, nq=16), n_terms=16384, hidden=256),
        # its network's training: mini-batches from a kept data set
        dict(name="train_1024x100", kind="train", rows=65536, batch=1024, steps=100, features=64, hidden=256),
        # a circuit seen once, from its gates to its expectations (the paper's hardware-efficient ansatz)
        dict(name="scan_hwea_100q", kind="scan", family="hwea", n=100),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["marginal", "marginal", "marginal", "zexpect", "zexpect", "batch", "both", "tencuts", "learned",
                       "train", "scan"])
    out = rng.choice(["host", "device"])
    if what == "marginal":
        c = rng.randint(1, 4)
        n = _log(rng, 8, 200)
        width = rng.randint(max(c, 2), min(12, n - 3))
        c = min(c, width)
        shots = rng.choice([0, 0, _log(rng, 100, 100_000), _log(rng, 100, 100_000)])
        if c == 4:
            shots = min(shots, 20_000)
        mirrored = rng.random() < 0.5
        flag = rng.choice(["", "", "", "", "sparse", "skip", "ml" if shots and not mirrored else ""])
        return _one("marginal", n, rng.randint(10, 60), width, str(c), rng.randint(1, 6), shots=shots,
                    nq=rng.randint(1, min(n, 16)), mirrored=mirrored, flag=flag, out=out,
                    precision=rng.choice(["fp64", "fp64", "fp32", "fp32x3"]))
    if what == "zexpect":
        c = rng.randint(1, 3)
        n = _log(rng, 20, 300)
        width = rng.randint(max(c, 3), 12)
        shots = rng.choice([0, _log(rng, 100, 100_000)])
        if n > 64:
            shots = min(shots, 10_000)
        return _one("zexpect", n, rng.randint(10, 60), width, str(c), rng.randint(1, 6), shots=shots,
                    strings=_log(rng, 1, 100), weight=rng.choice([0, 0, 6]), mirrored=rng.random() < 0.5, out=out,
                    flag=rng.choice(["", "", "settle" if shots else ""]))
    if what == "batch":
        circuits = _log(rng, 2, 200)
        return dict(kind="batch", circuits=circuits, shots=rng.choice([0, _log(rng, 100, 10_000), 10_000]), out=out)
    if what == "both":
        return _one("both", rng.randint(100, 400), rng.randint(15, 40), rng.randint(4, 8),
                    rng.choice(["2,2", "3,2", "3,3", "2,2,2"]), rng.randint(2, 10), nq=rng.randint(8, 16),
                    strings=_log(rng, 8, 100), topology="nn", p_cx=0.5, precision=rng.choice(["fp64", "fp32", "fp32x3"]),
                    out=out)
    if what == "tencuts":
        return _one("marginal", rng.randint(120, 300), rng.randint(20, 50), rng.randint(4, 6),
                    rng.choice(["3,3,2,2", "3,3,2", "3,3,3", "2,2,2,2"]), rng.randint(4, 12), nq=rng.randint(9, 16),
                    precision=rng.choice(["fp64", "fp32"]), flag=rng.choice(["", "", "sparse"]), out=out)
    if what == "learned":
        case = _one("learned", rng.randint(120, 300), rng.randint(20, 50), 5, rng.choice(["3,3,2,2", "3,3,2", "2,2,2"]),
                    rng.randint(4, 12), nq=rng.randint(8, 16), out=out)
        return dict(case, n_terms=_log(rng, 1000, 16384), hidden=rng.choice([64, 128, 256]))
    if what == "train":
        return dict(kind="train", rows=64 * _log(rng, 16, 1024), batch=64 * rng.randint(1, 16), steps=_log(rng, 10, 100),
                    features=64, hidden=rng.choice([64, 128, 192, 256]))
    family = rng.choice(["hwea", "qaoa", "phase"])
    n = _log(rng, 10, 100) if family == "hwea" else rng.randint(4, 20) if family == "qaoa" else rng.randint(5, 17)
    return dict(kind="scan", family=family, n=n)


# ---------------------------------------------------------------- inputs

def _circuit(case, seed):
    """(ops, cuts, requested qubits, Z-string masks) of a one-circuit case."""
    n, depth, width = case["n"], case["depth"], case["width"]
    counts = [int(c) for c in case["exits"].split(",")]
    rng = np.random.default_rng([seed, n, depth, 17])
    gap = n // len(counts)
    blocks = []
    for i, c in enumerate(counts):
        wires = list(range(i * gap, i * gap + width))
        blocks.append(W.Block(wires, wires[width - c:]))
    t_c = max(1, min(depth - 1, int(rng.integers(depth // 3, 2 * depth // 3 + 1))))
    ops, cuts = W.block_circuit(n, depth, blocks, t_c=t_c, p_cx=case["p_cx"], seed=seed, n_t=case["n_t"],
                                topology=case["topology"], mirrored=case["mirrored"])
    exits = {q for b in blocks for q in b.exits}
    nc = [q for b in blocks for q in b.wires if case["mirrored"] or q not in exits]
    taken = nc[:min(len(nc), max(1, case["nq"] // 2))] if case["nq"] else []
    others = [q for q in range(n) if q not in nc]
    near = sorted(others, key=lambda q: (min(abs(q - b.wires[-1]) for b in blocks), q))
    qubits = sorted((taken + near)[:case["nq"]])
    if len(qubits) < case["nq"]:
        qubits = sorted(qubits + [q for q in range(n) if q not in qubits][:case["nq"] - len(qubits)])
    masks = np.zeros((case["strings"], (n + 63) // 64), dtype=np.uint64)
    for i in range(case["strings"]):
        if case["weight"]:
            chosen = rng.choice(n, size=int(rng.integers(1, case["weight"] + 1)), replace=False)
        else:
            chosen = np.nonzero(rng.random(n) < 0.5)[0]
        for q in chosen:
            masks[i, q // 64] |= np.uint64(1 << (int(q) % 64))
    return ops, cuts, qubits, masks


def _scan(case, seed):
    make = {"hwea": W.hwea, "qaoa": W.qaoa_sk, "phase": W.phase_code}[case["family"]]
    return make(case["n"], seed=seed)


def _out(case, count):
    return torch.empty(count, dtype=torch.float64, device="cuda") if case["out"] == "device" else np.zeros(count)


def _parameters(F, H, seed):
    """He-initialised parameters of the F -> H -> H -> H -> 1 network, flat."""
    rng = np.random.default_rng([seed, 23])
    shapes = [(H, F), (H, H), (H, H), (1, H)]
    return np.concatenate([np.concatenate([(rng.normal(size=s) * math.sqrt(2.0 / s[1])).ravel(), np.zeros(s[0])])
                           for s in shapes]).astype(np.float32)


def _trained(F, H, cuts, seed):
    """Parameters that predict as a trained network does: unit 0 of every layer carries the sum of the cuts' log-shares
    (features 6c + 4 and 6c + 5), the others a small part of it."""
    rng = np.random.default_rng([seed, 31])
    W1, W2, W3, w4 = (rng.normal(size=s) * 0.02 / math.sqrt(s[1]) for s in ((H, F), (H, H), (H, H), (1, H)))
    W1[0] = 0.0
    for c in range(cuts):
        W1[0, 6 * c + 4:6 * c + 6] = -1.0
    for layer in (W2, W3):
        layer[0, 0] = 1.0
    w4[0, 0] = -1.0
    return np.concatenate([a for w, b in ((W1, H), (W2, H), (W3, H), (w4, 1))
                           for a in (w.ravel(), np.zeros(b))]).astype(np.float32)


def _training_set(case, seed):
    """Rows as the term model lays them out: per cut a one-hot digit, then two log-shares in [-1, 0]."""
    rng = np.random.default_rng([seed, 29])
    n, F = case["rows"], case["features"]
    cuts = F // 6
    x = np.zeros((n, F), dtype=np.float32)
    digits = rng.integers(0, 4, size=(n, cuts))
    shares = -rng.random((n, cuts, 2)).astype(np.float32) ** 2
    for c in range(cuts):
        x[np.arange(n), 6 * c + digits[:, c]] = 1.0
        x[:, 6 * c + 4:6 * c + 6] = shares[:, c]
    t = np.maximum(shares.sum(axis=(1, 2)) / 2, -1.0).astype(np.float32)
    return x, t


def prepare(case, seed):
    kind = case["kind"]
    ctx = cc.Context()
    state = dict(case=case, ctx=ctx, seed=seed)
    if kind in ("marginal", "zexpect", "both", "learned"):
        ops, cuts, qubits, masks = _circuit(case, seed)
        state.update(plan=cc.Plan(ctx, case["n"], ops, cuts), qubits=qubits, masks=masks)
        if kind != "zexpect":
            state["out"] = _out(case, 1 << case["nq"])
        if kind in ("zexpect", "both"):
            state["zout"] = _out(case, case["strings"])
        if kind == "learned":
            F = -(-6 * len(cuts) // 64) * 64
            state["net"] = cc.Mlp(ctx, F, case["hidden"])
            state["net"].set_params(_trained(F, case["hidden"], len(cuts), seed))
    elif kind == "batch":
        ws = [W.batching_circuit(seed % 1_000_003 * 256 + i, shots=case["shots"]) for i in range(case["circuits"])]
        plans = [cc.Plan(ctx, w.n, w.ops, w.cuts) for w in ws]
        state["batch"] = cc.Batch(ctx, plans, [w.qubits for w in ws], shots=case["shots"], seed=seed)
        state["out"] = _out(case, len(ws) << 16).reshape(len(ws), -1)
        state["outs"] = [row for row in state["out"]]
    elif kind == "scan":
        w = _scan(case, seed)
        state.update(ops=w.ops, n=w.n, qubits=w.qubits, masks=w.zmask_words())
    else:
        x, t = _training_set(case, seed)
        state["x"], state["t"] = torch.from_numpy(x).cuda().bfloat16(), torch.from_numpy(t).cuda()
        state["start"] = _parameters(case["features"], case["hidden"], seed)
        state["net"] = cc.Mlp(ctx, case["features"], case["hidden"])
    return state


# ---------------------------------------------------------------- one pass

def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "batch":
        state["batch"].run(state["outs"])
        return state["out"]
    if kind == "train":
        net = state["net"]
        net.set_params(state["start"])
        losses = net.train(state["x"], state["t"], batch=case["batch"], steps=case["steps"], lr=1e-3,
                           seed=state["seed"])
        return net.get_params(), losses
    if kind == "scan":
        plan = cc.Plan(state["ctx"], state["n"], state["ops"], cc.find_cuts(state["n"], state["ops"], 4))
        result = plan.marginal(state["qubits"]) if case["family"] == "phase" else plan.zexpect(state["masks"])
        plan.close()
        return result
    plan, qubits = state["plan"], state["qubits"]
    if kind == "learned":
        out, stderr = plan.learned_marginal(state["net"], qubits, case["n_terms"], seed=state["seed"], out=state["out"])
        return out, stderr
    options = dict(shots=case["shots"], seed=state["seed"], precision=PRECISION[case["precision"]],
                   flags=FLAGS[case["flag"]])
    if kind == "marginal":
        return plan.marginal(qubits, out=state["out"], **options)
    if kind == "zexpect":
        return plan.zexpect(state["masks"], out=state["zout"], **options)
    return (plan.marginal(qubits, out=state["out"], **options), plan.zexpect(state["masks"], out=state["zout"], **options))


# ---------------------------------------------------------------- what a pass cannot do without

def _sampling(variants, shots, measured):
    """Operations of drawing the shots: a share of the generator's words, one step per measurement, one count."""
    return variants * shots * (25.0 * -(-measured // 32) + measured + 1)


def work(case):
    """Circuit words read, outputs written; the shots drawn and the products of the smallest contraction."""
    kind = case["kind"]
    if kind == "batch":
        # circuits of 110 qubits and 40 layers on average, 55 Clifford variants of 12 measured qubits, 2^16 outputs
        circuits = case["circuits"]
        return {"bytes": circuits * (8.0 * (1 << 16) + 4.0 * 110 * 40),
                "flops": circuits * (_sampling(55, case["shots"], 12) + 2.0 * (1 << 16) * 30)}
    if kind == "train":
        H, F = case["hidden"], case["features"]
        weights = H * F + 2 * H * H + 4 * H + 1
        return {"bytes": case["steps"] * (2.0 * case["batch"] * F + 4.0 * case["batch"]) + 8.0 * weights,
                "flops": case["steps"] * 6.0 * case["batch"] * weights}
    if kind == "scan":
        n = case["n"] * (10 if case["family"] == "hwea" else case["n"] if case["family"] == "qaoa" else 4)
        out = 1 << (case["n"] - 1) if case["family"] == "phase" else case["n"]
        return {"bytes": 24.0 * n + 8.0 * out, "flops": 16.0 * n + 2.0 * out}
    counts = [int(c) for c in case["exits"].split(",")]
    k = sum(counts)
    n, depth = case["n"], case["depth"]
    outputs = (1 << case["nq"] if kind != "zexpect" else 0) + case["strings"]
    state_flops = len(counts) * (1 << case["width"]) * 14.0 * case["width"] * depth
    variants = (3 if case["mirrored"] else 4) ** k
    measured = min(n, case["nq"]) if kind == "marginal" else n
    flops = state_flops + 2.0 * outputs * (len(counts) + 1)
    if case["shots"]:
        flops += _sampling(variants, case["shots"], measured) + 2.0 * outputs * 4 ** max(counts)
    if kind == "learned":
        H = case["hidden"]
        flops += 2.0 * 4 ** k * (64 * H + 2 * H * H + H) + 2.0 * case["n_terms"] * outputs
    return {"bytes": 4.0 * n * depth + 8.0 * outputs, "flops": flops}


# ---------------------------------------------------------------- results in 64 bits

def _state_vector(n, ops):
    """|psi> of the uncut circuit, qubit q on axis q."""
    r = math.sqrt(0.5)
    phase = lambda a: np.array([[1, 0], [0, np.exp(1j * a)]])  # noqa: E731
    one = {"H": np.array([[r, r], [r, -r]]), "X": np.array([[0, 1], [1, 0]]), "Y": np.array([[0, -1j], [1j, 0]]),
           "Z": phase(np.pi), "S": phase(np.pi / 2), "SDG": phase(-np.pi / 2), "T": phase(np.pi / 4),
           "TDG": phase(-np.pi / 4)}
    psi = np.zeros((2,) * n, dtype=np.complex128)
    psi[(0,) * n] = 1.0
    for gate, a, b, theta in ops:
        if gate in ("CX", "CZ"):
            on = [slice(None)] * n
            on[a] = 1
            part = psi[tuple(on)]
            axis = b - (b > a)
            if gate == "CX":
                psi[tuple(on)] = np.flip(part, axis).copy()
            else:
                flip = [slice(None)] * (n - 1)
                flip[axis] = 1
                part[tuple(flip)] *= -1
        else:
            u = phase(theta) if gate == "RZ" else one[gate]
            psi = np.moveaxis(np.tensordot(u, psi, axes=(1, a)), 0, a)
    return psi


def _draw_rows(seed, steps, batch, n):
    """Mini-batch rows: word 0 and so on of Philox4x32-10 at counter (i, s, 0x4D4C5000, 0), modulo n."""
    i, s = np.meshgrid(np.arange(batch, dtype=np.uint64), np.arange(steps, dtype=np.uint64))
    c = [i, s, np.full_like(i, 0x4D4C5000), np.zeros_like(i)]
    key = [np.uint64(seed & 0xFFFFFFFF), np.uint64(seed >> 32 & 0xFFFFFFFF)]
    low = np.uint64(0xFFFFFFFF)
    for _ in range(10):
        p, q = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(q >> np.uint64(32)) ^ c[1] ^ key[0], q & low, (p >> np.uint64(32)) ^ c[3] ^ key[1], p & low]
        key = [(key[0] + np.uint64(0x9E3779B9)) & low, (key[1] + np.uint64(0xBB67AE85)) & low]
    return c


def _train(case, seed):
    x, t = _training_set(case, seed)
    x = torch.from_numpy(x).bfloat16().double().numpy()
    F, H = case["features"], case["hidden"]
    p = _parameters(F, H, seed).astype(np.float64)
    n, batch = case["rows"], case["batch"]
    words = _draw_rows(seed, case["steps"], batch, n)
    cut = np.cumsum([H * F, H, H * H, H, H * H, H, H])
    m, v, losses = np.zeros_like(p), np.zeros_like(p), []
    for step in range(case["steps"]):
        rows = (words[0][step] % np.uint64(n)).astype(np.int64) if batch != n else np.arange(n)
        W1, b1, W2, b2, W3, b3, w4, b4 = np.split(p, cut)
        W1, W2, W3 = W1.reshape(H, F), W2.reshape(H, H), W3.reshape(H, H)
        h0 = x[rows]
        h1 = np.maximum(h0 @ W1.T + b1, 0)
        h2 = np.maximum(h1 @ W2.T + b2, 0)
        h3 = np.maximum(h2 @ W3.T + b3, 0)
        d = h3 @ w4 + b4 - t[rows].astype(np.float64)
        losses.append(np.mean(d * d))
        d = 2 * d / batch
        g4, g = d @ h3, np.outer(d, w4) * (h3 > 0)
        parts = [np.concatenate([(g.T @ h2).ravel(), g.sum(0)])]
        g = (g @ W3) * (h2 > 0)
        parts.insert(0, np.concatenate([(g.T @ h1).ravel(), g.sum(0)]))
        g = (g @ W2) * (h1 > 0)
        parts.insert(0, np.concatenate([(g.T @ h0).ravel(), g.sum(0)]))
        grad = np.concatenate(parts + [g4, [d.sum()]])
        m, v = 0.9 * m + 0.1 * grad, 0.999 * v + 0.001 * grad * grad
        p = p - 1e-3 * (m / (1 - 0.9 ** (step + 1))) / (np.sqrt(v / (1 - 0.999 ** (step + 1))) + 1e-8)
    return p, np.array(losses)


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        if case["steps"] * case["batch"] * case["hidden"] ** 2 > 1e10:
            return None
        return _train(case, seed)
    if kind == "scan":
        w = _scan(case, seed)
        n, ops, qubits, masks = w.n, w.ops, w.qubits, w.zmask_words()
        marginal = case["family"] == "phase"
    elif kind in ("marginal", "zexpect") and not case["shots"]:
        n = case["n"]
        ops, _, qubits, masks = _circuit(case, seed)
        marginal = kind == "marginal"
    else:
        return None
    if n > 18:
        return None
    p = np.abs(_state_vector(n, ops)) ** 2
    if marginal:
        rest = tuple(q for q in range(n) if q not in qubits)
        p = p.sum(axis=rest)
        order = [sorted(qubits).index(q) for q in qubits]
        return np.ascontiguousarray(np.transpose(p, order[::-1])).ravel()  # bit i = qubits[i]
    sign = np.array([1.0, -1.0])
    out = []
    for row in masks:
        e = p
        for q in range(n - 1, -1, -1):
            e = e @ (sign if int(row[q // 64]) >> (q % 64) & 1 else np.ones(2))
        out.append(float(e))
    return np.array(out)
