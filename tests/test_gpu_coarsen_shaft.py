"""Merge errors of the light coarsening where the wavefront-shared shadow test
can go wrong: no spheres, a partly filled group of spheres, more than 64 groups,
and so many spheres above the points that the list of candidates overflows and
the traversal takes over; with draws enough to open the top of the tree (its
lights evaluated once per row) and too few to open it.  Against the FP64 oracle,
within the bound of every merge-error test: 1e-4 relative + 1e-5 of the largest
(FP32 shading), nodes with an ambiguous visibility excluded."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import coarsen as C  # noqa: E402
from oracle import render as orender  # noqa: E402
from paper_2202_12567_amd import api  # noqa: E402
from scenegen import make_scene  # noqa: E402

SEED = 6
SLICES = (1, 12)


def spheres(kind):
    rng = np.random.default_rng(17)
    if kind == "none":
        n, lo, hi, r = 0, 0, 0, (0.01, 0.02)
    elif kind == "partial group":
        n, lo, hi, r = 33, 0.05, 0.2, (0.02, 0.08)
    elif kind == "many groups":
        n, lo, hi, r = 2100, 0.12, 0.24, (0.004, 0.02)
    else:
        n, lo, hi, r = 700, 0.21, 0.24, (0.01, 0.03)
    side = (0.35, 0.65) if kind == "overflow" else (0.0, 1.0)
    f = np.float32
    return dict(cx=rng.uniform(*side, n).astype(f), cy=rng.uniform(*side, n).astype(f),
                cz=rng.uniform(lo, hi, n).astype(f), r=rng.uniform(*r, n).astype(f))


@pytest.mark.parametrize("kind", ["none", "partial group", "many groups", "overflow"])
@pytest.mark.parametrize("K", [600, 4096])
def test_merge_errors(kind, K):
    sc = dataclasses.replace(make_scene("tiny", SEED), spheres=spheres(kind))
    prm = api.default_params(seed=SEED, pass1_ppm=0, pass2_ppm=20000, max_iter=2, fixed_iters=True)
    dev = torch.device("cuda", 0)
    ctx = api.Context(0)
    ctx.set_occluders(sc.spheres)
    ds = api.DeviceScene(sc, dev)
    plan = api.Plan(sc, prm, api.Coarsening(K, 128))
    ws = api.workspace(plan, dev)
    api.render(ctx, plan, ds, prm, ws)
    ng = sc.n_clusters
    eps = api.region_view(plan, ws, "NODE_EPS", torch.float32).cpu().numpy().reshape(sc.n_slices, ng - 1)
    table = C.scene_table(sc, SEED)
    oprm = orender.Params(seed=SEED, pass1_ppm=0, pass2_ppm=20000, max_iter=2, fixed_iters=True)
    shadowed = 0
    for s in SLICES:
        co = C.coarsen_slice(sc, table, s, SEED, C.CoarsenParams(pixels=K), 128, oprm)
        nodes = np.array(sorted(co["eps"]), np.int64)
        o = np.array([co["eps"][f] for f in nodes])
        amb = np.array([f in co["ambiguous_nodes"] for f in nodes])
        g = eps[s, nodes - ng]
        bad = (np.abs(g - o) > 1e-4 * o + 1e-5 * max(float(o.max()), 1e-30)) & ~amb
        assert not bad.any(), (s, nodes[bad][:10])
        assert amb.mean() < 0.2
        shadowed += int((o > 0).sum())
    assert shadowed > 0
