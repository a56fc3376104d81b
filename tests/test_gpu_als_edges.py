"""Masked ALS at the edges of its kernels' tiling (row groups of 16 and 64,
column groups of 16 and 256, 8 at rank 32; sample blocks of 8 and 16), with a
fully sampled column, a column and a row without samples, and an odd and an
even iteration count (the two X buffers), against the FP64 oracle on the same
samples.  1e-3 per slice: the per-slice bar of every completion test, three
orders above the FP32 rounding of the Grams."""
import types

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import render as orender  # noqa: E402
from oracle.sampling import count_from_ppm  # noqa: E402
from paper_2202_12567_amd import api  # noqa: E402

SEED = 9
PPM = 350000


def samples_of(m, n, rng):
    """Distinct entries: column 0 whole, the last column and (m > 2) the last row empty, the rest at random."""
    N1 = count_from_ppm(PPM, m * n)
    ok = np.ones((m, n), bool)
    if m > 2 and n > 2:
        ok[-1] = ok[:, -1] = False
    first = np.arange(m)[ok[:, 0]] * n
    rest = np.setdiff1d(np.flatnonzero(ok.ravel()), first)
    e = np.concatenate([first, rng.permutation(rest)])[:N1]
    assert e.shape[0] == N1
    return rng.permutation(e)


@pytest.mark.parametrize("iters", [6, 7])
@pytest.mark.parametrize("m,n,q", [(3, 1, 1), (16, 16, 16), (17, 257, 16), (64, 33, 8), (65, 40, 32), (33, 260, 4),
                                   (1100, 12, 12)])
def test_als_tile_edges(m, n, q, iters):
    rng = np.random.default_rng(m * 1000 + n)
    plan_of = types.SimpleNamespace(n_slices=1, n_clusters=n, pt_offsets=np.array([0, m], np.int32),
                                    cl_offsets=np.array([0, n], np.int32), rank=np.array([q], np.int32))
    prm = api.default_params(seed=SEED, pass1_ppm=PPM, pass2_ppm=0, max_iter=iters, fixed_iters=True, als=True)
    dev = torch.device("cuda", 0)
    ctx = api.Context(0)
    plan = api.Plan(plan_of, prm)
    ws = api.workspace(plan, dev)
    e = samples_of(m, n, rng)
    ii, jj = e // n, e % n
    vals = rng.uniform(0.1, 2.0, (e.shape[0], 3)).astype(np.float32)
    keys = ((ii << 16) | jj).astype(np.uint32).view(np.int32)
    api.region_view(plan, ws, "OMEGA1", torch.int32)[: e.shape[0]] = torch.as_tensor(keys, device=dev)
    api.region_view(plan, ws, "VAL1", torch.float32)[: 3 * e.shape[0]] = torch.as_tensor(vals.ravel(), device=dev)
    pt = torch.arange(m, dtype=torch.int32, device=dev)
    rad = api.stage_adm(ctx, plan, prm, pt, ws, n_points=m).double().cpu().numpy()
    st = api.read_stats(ctx, plan, ws)
    want, n_it, err, _, _ = orender.complete_and_render(
        m, n, q, ii, jj, vals.astype(np.float64), SEED, 0,
        orender.Params(seed=SEED, max_iter=iters, fixed_iters=True, method="als", lam=0.01))
    assert int(st["iters"][0]) == n_it == iters
    assert abs(float(st["resid"][0]) - err) <= 1e-3 * err + 1e-6
    assert orender.relative_rmse(rad, want) <= 1e-3
