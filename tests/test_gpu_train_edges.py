"""Gradients and a training step of the proposal network at the edges of the
training kernels' row tiles (32 rows per wavefront, 128 and 256 per workgroup,
blocks of 16 and 64 in the dW2 product, several tiles per workgroup), with a
scratch that is only float-aligned, against the FP64 oracle.  1e-2 relative per
tensor: a bfloat16 rounding that falls the other way moves one activation by
2^-8."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import mlp as omlp  # noqa: E402
from paper_2202_12567_amd import api  # noqa: E402

DEV = torch.device("cuda", 0)


def inputs(rows):
    rng = np.random.default_rng(rows)
    h, k = 128, 12
    pv = np.concatenate([rng.normal(0, np.sqrt(2 / k), h * k), rng.normal(0, 0.1, h),
                         rng.normal(0, np.sqrt(2 / h), h * h), rng.normal(0, 0.1, h),
                         rng.normal(0, np.sqrt(1 / h), h), rng.normal(0, 0.1, 1)]).astype(np.float32)
    return rng, pv, rng.uniform(-1, 2, (rows, k)).astype(np.float32)


def close(got, want):
    gu, wu = omlp.unflatten(got), omlp.unflatten(want)
    for k in omlp.PARAM_ORDER:
        assert np.linalg.norm(gu[k] - wu[k]) <= 1e-2 * np.linalg.norm(wu[k]) + 1e-12, k


@pytest.mark.parametrize("rows", [1, 31, 33, 64, 127, 257, 4099])
@pytest.mark.parametrize("shift", [0, 4])
def test_gradient_at_tile_edges(rows, shift):
    rng, pv, F = inputs(rows)
    dy = rng.normal(0, 1, rows).astype(np.float32)
    ctx = api.Context(0)
    scratch = torch.empty(api.mlp_scratch(rows, DEV).numel() + 4, dtype=torch.uint8, device=DEV)[shift:]
    t = [torch.as_tensor(a).to(DEV) for a in (pv, F, dy)]
    g = api.mlp_grad(ctx, *t, scratch=scratch).cpu().numpy()
    _, c = omlp.forward(omlp.unflatten(pv), F, rounding=True)
    close(g, omlp.flatten(omlp.backward(c, dy)))


def test_several_tiles_per_workgroup():
    """70,003 rows: every backward workgroup walks more than one tile.  The gradient is linear in the rows, so the
    sum of the gradients of the two halves is the reference."""
    rows, cut = 70003, 30011
    rng, pv, F = inputs(rows)
    dy = rng.normal(0, 1, rows).astype(np.float32)
    ctx = api.Context(0)
    p = torch.as_tensor(pv).to(DEV)
    f, d = torch.as_tensor(F).to(DEV), torch.as_tensor(dy).to(DEV)
    whole = api.mlp_grad(ctx, p, f, d).double()
    parts = sum(api.mlp_grad(ctx, p, f[a:b].contiguous(), d[a:b].contiguous()).double() for a, b in ((0, cut), (cut, rows)))
    # FP32 sums over 7e4 rows in another order: 6e-8 sqrt(7e4) of the summed magnitudes
    assert float((whole - parts).norm() / whole.norm()) < 1e-4


def test_step_leaves_gradient_logits_and_slopes_in_scratch():
    """The documented start of the scratch: gradient, logits y, softmax(y) - pstar."""
    groups = [0, 5, 70, 131]
    rows = groups[-1]
    rng, pv, F = inputs(rows)
    p = rng.uniform(0.1, 1, rows)
    for a, b in zip(groups[:-1], groups[1:]):
        p[a:b] /= p[a:b].sum()
    ctx = api.Context(0)
    t = [torch.as_tensor(a).to(DEV) for a in (pv, np.zeros_like(pv), np.zeros_like(pv))]
    scratch, loss = api.mlp_scratch(rows, DEV), torch.zeros(1, device=DEV)
    api.mlp_train_step(ctx, *t, 1, 1e-3, torch.as_tensor(F).to(DEV), torch.as_tensor(p.astype(np.float32)).to(DEV),
                       torch.as_tensor(np.array(groups, np.int32)).to(DEV), scratch, loss)
    out = scratch[:4 * (api.mlp_param_count() + 2 * rows)].view(torch.float32).cpu().numpy()
    g, y, dy = np.split(out, [api.mlp_param_count(), api.mlp_param_count() + rows])
    yo, c = omlp.forward(omlp.unflatten(pv), F, rounding=True)
    assert np.abs(y - yo).max() <= 1e-2 * np.abs(yo).max()
    want = np.concatenate([np.exp(y[a:b] - y[a:b].max()) / np.exp(y[a:b] - y[a:b].max()).sum()
                           for a, b in zip(groups[:-1], groups[1:])]) - p
    assert np.abs(dy - want).max() <= 1e-5
    close(g, omlp.flatten(omlp.backward(c, dy)))
