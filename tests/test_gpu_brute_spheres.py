"""The brute-force column sum against spheres at the edges of its split (segments
of 4,096 outputs, runs of 64 neighbouring points, wavefronts that share a run's
lights) and of its shared shadow test (no spheres, a partly filled group, more
than 64 groups, lists that overflow), with repeated points, points all in one
place and points too far away for a box.  Against the FP64 sum of the same FP32
entries from the per-pair kernel, whose every shadow ray walks the BVH: equal up
to the rounding of at most 300 FP64 additions, 300 x 2^-53 < 1e-13 of the sum."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2202_12567_amd import api  # noqa: E402
from scenegen import make_scene  # noqa: E402
from test_gpu_coarsen_shaft import spheres  # noqa: E402

SEED = 6


@pytest.mark.parametrize("n_out,n_lights,kind,points", [
    (1, 300, "partial group", "drawn"), (63, 65, "many groups", "drawn"), (64, 1, "partial group", "drawn"),
    (65, 300, "overflow", "drawn"), (1024, 129, "none", "drawn"), (1025, 64, "many groups", "drawn"),
    (4096, 63, "overflow", None), (4097, 65, "partial group", "drawn"), (9000, 33, "many groups", "drawn"),
    (700, 300, "many groups", "one place"), (700, 300, "partial group", "far")])
def test_sums_of_the_pairs(n_out, n_lights, kind, points):
    sc = make_scene("tiny", SEED)
    if points == "one place":
        sc = dataclasses.replace(sc, points={k: np.repeat(v[77:78], v.shape[0]) for k, v in sc.points.items()})
    elif points == "far":
        px = sc.points["px"].copy()
        px[::5] = 3e18
        sc = dataclasses.replace(sc, points={**sc.points, "px": px})
    dev = torch.device("cuda", 0)
    prm = api.default_params()
    ctx = api.Context(0)
    ctx.set_occluders(spheres(kind))
    ds = api.DeviceScene(sc, dev)
    lights = {k: v[:n_lights].contiguous() for k, v in ds.vpl.items()}
    rng = np.random.default_rng(n_out)
    pid = None if points is None else torch.as_tensor(rng.integers(0, sc.m, n_out, dtype=np.int32), device=dev)
    got = api.brute_force(ctx, ds, lights, prm, pid, n_out=n_out)
    p = torch.arange(n_out, dtype=torch.int32, device=dev) if pid is None else pid
    pairs = api.eval_pairs(ctx, ds, lights, p.repeat_interleave(n_lights).contiguous(),
                           torch.arange(n_lights, dtype=torch.int32, device=dev).repeat(n_out), prm)
    want = pairs.double().reshape(n_out, n_lights, 3).sum(1)
    assert float(want.sum()) > 0
    assert bool(((got - want).abs() <= 1e-13 * want).all())
