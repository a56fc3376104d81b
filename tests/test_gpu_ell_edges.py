"""The LDS-resident completion at the edges of its work split (items of 16
column parts, steps of 4 samples, groups of 64 parts, parts of at most 64
samples, padded ranks): columns of every length around those bounds, an empty
and a full one, in slices with fewer items than wavefronts and with many,
against the FP64 oracle on the same samples.  1e-3 per slice: the per-slice bar
of every completion test, three orders above the FP32 rounding of an iterate."""
import types

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import render as orender  # noqa: E402
from oracle.sampling import count_from_ppm  # noqa: E402
from paper_2202_12567_amd import api  # noqa: E402

SEED = 6
ITERS = 9
LENGTHS = [0, 1, 3, 4, 5, 8, 9, 63, 64, 65, 127, 128, 129]


@pytest.mark.parametrize("m,n,q,threads", [(140, 15, 12, 1024), (140, 16, 8, 1024), (131, 17, 4, 1024),
                                           (200, 63, 16, 512), (150, 65, 5, 1024), (300, 129, 13, 1024),
                                           (1000, 255, 16, 1024), (260, 1041, 8, 512)])
def test_parts_items_steps(m, n, q, threads):
    rng = np.random.default_rng(m + n)
    lens = np.resize(np.array(LENGTHS + [m]), n)
    ii = np.concatenate([rng.permutation(m)[:k] for k in lens])
    jj = np.repeat(np.arange(n), lens)
    ppm = int(round(ii.size / (m * n) * 1e6))
    N1 = count_from_ppm(ppm, m * n)                  # the rate rounds to a neighbouring count
    if N1 < ii.size:
        ii, jj = ii[:N1], jj[:N1]
    free = np.setdiff1d(np.arange(m * n), ii * n + jj)
    more = free[free % n != 0][:N1 - ii.size]        # column 0 stays empty
    ii, jj = np.concatenate([ii, more // n]), np.concatenate([jj, more % n])
    shape = types.SimpleNamespace(n_slices=1, n_clusters=n, pt_offsets=np.array([0, m], np.int32),
                                  cl_offsets=np.array([0, n], np.int32), rank=np.array([q], np.int32))
    prm = api.default_params(seed=SEED, pass1_ppm=ppm, pass2_ppm=0, max_iter=ITERS, fixed_iters=True)
    dev = torch.device("cuda", 0)
    ctx = api.Context(0)
    plan = api.Plan(shape, prm)
    assert plan.slice_info(0)["adm_in_lds"]
    api.set_tune(plan, adm_threads=threads)
    ws = api.workspace(plan, dev)
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
