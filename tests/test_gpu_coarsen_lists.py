"""The coarsening's walks against each other, bit for bit.  More than 16,384 spheres turn the wavefront-shared lists
off, so spheres that no segment can meet, far below the scene, give the traversal's answer; half the slices are too
few draws for the level-by-level walk and take the one of a path per thread."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2202_12567_amd import api  # noqa: E402
from scenegen import make_scene, scene_sample  # noqa: E402

SEED = 6
DEV = torch.device("cuda", 0)


def below(sph, count):
    rng = np.random.default_rng(2)
    f = np.float32
    far = dict(cx=rng.uniform(0, 1, count), cy=rng.uniform(0, 1, count), cz=rng.uniform(-11, -10, count),
               r=np.full(count, 1e-3))
    return {k: np.concatenate([sph[k], far[k].astype(f)]) for k in ("cx", "cy", "cz", "r")}


def merge_errors(sc, spheres, K):
    prm = api.default_params(seed=SEED, pass1_ppm=0, pass2_ppm=20000, max_iter=2, fixed_iters=True)
    ctx = api.Context(0)
    ctx.set_occluders(spheres)
    ds = api.DeviceScene(sc, DEV)
    plan = api.Plan(sc, prm, api.Coarsening(K, 128))
    ws = api.workspace(plan, DEV)
    api.render(ctx, plan, ds, prm, ws)
    return api.region_view(plan, ws, "NODE_EPS", torch.int32).clone()


@pytest.mark.parametrize("K", [600, 4096, 32768])
@pytest.mark.parametrize("normal", [None, np.inf, -np.inf, 1e30, np.nan])
def test_equals_the_traversal(K, normal):
    """With normals that put a shadow segment's origin beyond any box, in one row of every 50."""
    sc = make_scene("tiny", SEED)
    if normal is not None:
        pts = {k: np.array(v) for k, v in sc.points.items()}
        for k, axis in enumerate(("nx", "ny", "nz")):
            pts[axis][sc.pt_ids[k * 17::50]] = normal
        sc = dataclasses.replace(sc, points=pts)
    lists, walk = (merge_errors(sc, below(sc.spheres, extra), K) for extra in (0, 17000))
    assert int((lists != 0).sum()) > 500
    assert torch.equal(lists, walk)


def occluders(kind):
    rng = np.random.default_rng(17)
    n, side, z, r = {"none": (0, (0, 1), (0, 1), (0.1, 0.2)), "own": (0, (0, 1), (0, 1), (0.1, 0.2)),
                     "65 groups": (2080, (0, 1), (0.12, 0.24), (0.004, 0.02)),
                     "overflow, staged": (700, (0.35, 0.65), (0.21, 0.24), (0.01, 0.03)),
                     "overflow": (1600, (0.35, 0.65), (0.21, 0.24), (0.006, 0.018))}[kind]
    f = np.float32
    return dict(cx=rng.uniform(*side, n).astype(f), cy=rng.uniform(*side, n).astype(f),
                cz=rng.uniform(*z, n).astype(f), r=rng.uniform(*r, n).astype(f))


@pytest.mark.parametrize("kind,K", [("own", 32768), ("65 groups", 32768), ("overflow, staged", 32768), ("overflow", 32768),
                                    ("overflow", 70001), ("triangles", 32768), ("none", 262144)])
def test_levels_equal_the_walk_per_thread(kind, K):
    """16 slices of 32,768 draws are 2^19, from where the walk goes level by level (2^22 without occluders)."""
    sc = make_scene("tri" if kind == "triangles" else "tiny", SEED)
    sph = sc.spheres if kind in ("own", "triangles") else occluders(kind)
    few = merge_errors(scene_sample(sc, list(range(8))), sph, K)
    many = merge_errors(sc, sph, K)
    assert int((few != 0).sum()) > 500
    assert torch.equal(many[:few.shape[0]], few)


def coarsen_ms(sc, spheres, K):
    prm = api.default_params(seed=SEED, pass1_ppm=0, pass2_ppm=20000, max_iter=2, fixed_iters=True)
    ctx = api.Context(0)
    ctx.set_occluders(spheres)
    ds = api.DeviceScene(sc, DEV)
    plan = api.Plan(sc, prm, api.Coarsening(K, 128))
    ws, rad = api.workspace(plan, DEV), torch.empty((sc.m, 3), device=DEV)
    best = []
    for _ in range(6):
        api.profile_begin(ctx, 1)
        api.render(ctx, plan, ds, prm, ws, rad)
        torch.cuda.synchronize()
        best.append(api.profile_end(ctx)[0]["coarsen"])
    return min(best)


@pytest.mark.parametrize("K", [600, 4096, 32768])
def test_lists_that_overflow_cost_little(K):
    """Spheres so dense that no wavefront's list holds them: at most half as long again as the same walk without
    lists (every list tried and then traversed all the same took 1.8 to 2.3 times as long)."""
    sc = make_scene("tiny", SEED)
    rng = np.random.default_rng(17)
    f = np.float32
    n = 16000
    dense = dict(cx=rng.uniform(0, 1, n).astype(f), cy=rng.uniform(0, 1, n).astype(f),
                 cz=rng.uniform(0.05, 0.24, n).astype(f), r=rng.uniform(0.005, 0.02, n).astype(f))
    assert coarsen_ms(sc, dense, K) <= 1.5 * coarsen_ms(sc, below(dense, 1000), K)
