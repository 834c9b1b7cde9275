"""Edges of the training kernels: batches of one 64-row piece, of a last
half-staged piece and of a partly filled 256-row chunk; the narrowest and
widest layers; data sets whose rows are not 16-byte aligned; fp32 rows.

Gradients against the fp64 oracle at the same bf16-rounded weights and
inputs.  Tolerance: activations and pre-activation gradients are stored in
bf16 (relative rounding 2^-9 each), six roundings deep at most along a path
and averaged over the batch; narrow nets over few rows average least and
are held to cosine >= 0.995 and relative error <= 1e-1 per tensor, the bar
of the existing gradient test at those shapes.  The other comparisons are
bit for bit."""
import numpy as np
import pytest

import paper_2303_10788_amd as cc
from oracle import mlp as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    return cc.Context()


def _bf16(a):
    import torch
    return torch.tensor(np.asarray(a, dtype=np.float32)).to(torch.bfloat16).to(torch.float32).numpy()


def _case(F, H, rows, seed):
    import torch
    rng = np.random.default_rng([seed, F, H, rows])
    params = [(_bf16(W).astype(np.float64), _bf16(b + 0.05 * rng.normal(size=b.shape)).astype(np.float64))
              for W, b in O.init_params(F, H, seed)]
    x = _bf16(rng.normal(size=(rows, F)))
    t = rng.normal(size=rows).astype(np.float32)
    return params, x, t, torch.tensor(x).to(torch.bfloat16).cuda(), torch.tensor(t).cuda()


EDGES = [(64, 64, 64), (256, 64, 192), (64, 256, 320), (192, 128, 1088), (256, 256, 64), (64, 256, 1216)]
PAIRS = [(F, H, 128) for F in (64, 128, 192, 256) for H in (64, 128, 192, 256)]  # one kernel each


@pytest.mark.parametrize("F,H,rows", EDGES + PAIRS)
def test_gradients_at_edges(ctx, F, H, rows):
    print(f"gradients F={F} H={H} rows={rows}", flush=True)
    params, x, t, xd, td = _case(F, H, rows, 3)
    net = cc.Mlp(ctx, F, H)
    net.set_params(cc.mlp_pack(params))
    g, loss = net.gradients(xd, td)
    ref_loss, ref = O.loss_and_grads(params, x.astype(np.float64), t.astype(np.float64))
    assert abs(loss - ref_loss) <= 2e-2 * ref_loss
    for (gw, gb), (rw, rb) in zip(cc.mlp_unpack(g.astype(np.float64), F, H), ref):
        for a, r in ((gw, rw), (gb, rb)):
            a, r = np.ravel(a), np.ravel(r)
            assert a @ r >= 0.995 * np.linalg.norm(a) * np.linalg.norm(r)
            assert np.linalg.norm(a - r) <= 1e-1 * np.linalg.norm(r)


@pytest.mark.parametrize("F,H,rows,batch", [(64, 64, 192, 64), (128, 192, 960, 448), (64, 256, 512, 512)])
def test_rows_not_aligned(ctx, F, H, rows, batch):
    """The same data two bytes off a 16-byte boundary trains to the same parameters."""
    import torch
    print(f"unaligned rows F={F} H={H} rows={rows} batch={batch}", flush=True)
    params, _, _, xd, td = _case(F, H, rows, 5)
    off = torch.empty(rows * F + 1, dtype=torch.bfloat16, device="cuda")[1:].view(rows, F)
    off.copy_(xd)
    assert off.data_ptr() % 16 and xd.data_ptr() % 16 == 0
    got = []
    for data in (xd, off):
        net = cc.Mlp(ctx, F, H)
        net.set_params(cc.mlp_pack(params))
        losses = net.train(data, td, batch=batch, steps=3, lr=1e-3, seed=9)
        got.append((net.get_params(), losses))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])


def test_fp32_rows_equal_rounded_rows(ctx):
    """train_step rounds fp32 rows itself: two steps equal train() over the rounded rows in order, bit for bit."""
    import torch
    F, H, rows = 64, 128, 320
    print("fp32 rows", flush=True)
    params, _, _, _, td = _case(F, H, rows, 7)
    xf = torch.randn(rows, F, generator=torch.Generator().manual_seed(1)).cuda()
    a, b = cc.Mlp(ctx, F, H), cc.Mlp(ctx, F, H)
    for net in (a, b):
        net.set_params(cc.mlp_pack(params))
    first = [a.train_step(xf, td), a.train_step(xf, td)]
    losses = b.train(xf.to(torch.bfloat16), td, batch=rows, steps=2, lr=1e-3, seed=0)
    assert np.array_equal(np.float32(first), losses)
    assert np.array_equal(a.get_params(), b.get_params())
