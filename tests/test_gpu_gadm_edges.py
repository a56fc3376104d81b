"""The global-memory completion at the edges of its tiling (64-row blocks,
64-column blocks of the small-frame rule, 16-component Gram tiles, padded
ranks), a column of more samples than a lane group takes and an empty column,
against the FP64 oracle on the same samples at an odd iteration count (the
second X buffer).  1e-3 per slice: the per-slice bar of every completion test,
three orders above the FP32 rounding of the Grams."""
import types

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import render as orender  # noqa: E402
from oracle.sampling import count_from_ppm  # noqa: E402
from paper_2202_12567_amd import api  # noqa: E402

SEED = 4
ITERS = 9


@pytest.mark.parametrize("m,n,q,ppm", [(32, 32, 32, 500000), (65, 64, 32, 300000), (64, 65, 20, 300000),
                                       (129, 257, 17, 200000), (1300, 130, 32, 150000), (1200, 63, 16, 150000),
                                       (2500, 66, 8, 80000), (4700, 40, 4, 60000), (4801, 9, 3, 100000)])
def test_global_memory_tiles(m, n, q, ppm):
    rng = np.random.default_rng(m + n)
    shape = types.SimpleNamespace(n_slices=1, n_clusters=n, pt_offsets=np.array([0, m], np.int32),
                                  cl_offsets=np.array([0, n], np.int32), rank=np.array([q], np.int32))
    prm = api.default_params(seed=SEED, pass1_ppm=ppm, pass2_ppm=0, max_iter=ITERS, fixed_iters=True)
    dev = torch.device("cuda", 0)
    ctx = api.Context(0)
    plan = api.Plan(shape, prm)
    assert not plan.slice_info(0)["adm_in_lds"]
    ws = api.workspace(plan, dev)
    N1 = count_from_ppm(ppm, m * n)
    ok = np.ones((m, n), bool)
    ok[:, -1] = False                                        # an empty column
    first = (np.arange(m) * n)[:N1 // 2]                     # a long one
    e = np.concatenate([first, rng.permutation(np.setdiff1d(np.flatnonzero(ok.ravel()), first))])[:N1]
    ii, jj = e // n, e % n
    vals = rng.uniform(0.1, 2.0, (N1, 3)).astype(np.float32)
    api.region_view(plan, ws, "OMEGA1", torch.int32)[:N1] = torch.as_tensor(
        ((ii << 16) | jj).astype(np.uint32).view(np.int32), device=dev)
    api.region_view(plan, ws, "VAL1", torch.float32)[: 3 * N1] = torch.as_tensor(vals.ravel(), device=dev)
    pt = torch.arange(m, dtype=torch.int32, device=dev)
    rad = api.stage_adm(ctx, plan, prm, pt, ws, n_points=m).double().cpu().numpy()
    want, _, err, _, _ = orender.complete_and_render(
        m, n, q, ii, jj, vals.astype(np.float64), SEED, 0,
        orender.Params(seed=SEED, max_iter=ITERS, fixed_iters=True))
    st = api.read_stats(ctx, plan, ws)
    assert int(st["iters"][0]) == ITERS
    assert abs(float(st["resid"][0]) - err) <= 1e-3 * err + 1e-6
    assert orender.relative_rmse(rad, want) <= 1e-3
