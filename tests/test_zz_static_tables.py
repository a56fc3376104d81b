"""The static workspace's limit leaves out the tables that only save time: a
coarsened frame whose workspace exceeds 64 MiB only by its top table still runs
there, one whose top table would not fit beside it is planned without it, and
one that is too large by itself stays refused.  Each frame that runs equals the
frame of the same plan on a caller's workspace, bit for bit."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2202_12567_amd import _native as N  # noqa: E402
from paper_2202_12567_amd import api  # noqa: E402
from scenegen import make_scene  # noqa: E402

MIB = 1 << 20


@pytest.fixture(scope="module")
def scene():
    sc = make_scene("tiny", 6)
    twice = {k: np.concatenate([v, v]) for k, v in sc.points.items()}      # 32 slices of 256 rows
    return dataclasses.replace(
        sc, points=twice, pt_ids=np.concatenate([sc.pt_ids, sc.pt_ids + sc.m]).astype(np.int32),
        pt_offsets=(np.arange(33) * 256).astype(np.int32), rank=np.tile(sc.rank, 2),
        cl_offsets=(np.arange(33) * sc.n_clusters).astype(np.int32), cl_ids=np.tile(sc.cl_ids, 2))


@pytest.mark.parametrize("K,n_max,fits", [(16384, 64, "with its tables"), (32768, 64, "without the top table"),
                                          (32768, 128, "not")])
def test_coarsened_frame(scene, K, n_max, fits):
    dev = torch.device("cuda", 0)
    prm = api.default_params(seed=6, pass1_ppm=0, pass2_ppm=20000, max_iter=5, fixed_iters=True)
    ctx = api.Context(0)
    ctx.set_occluders(scene.spheres)
    ds = api.DeviceScene(scene, dev)
    plan = api.Plan(scene, prm, api.Coarsening(K, n_max))
    assert (plan.workspace_bytes > 64 * MIB) == (fits != "without the top table")
    if fits == "not":
        with pytest.raises(N.VplmcError) as e:
            api.render_static(ctx, plan, ds, prm)
        assert e.value.code == N.EINVAL
        return
    ref = api.render(ctx, plan, ds, prm, api.workspace(plan, dev)).clone()
    got = torch.full((scene.m, 3), -1.0, dtype=torch.float32, device=dev)
    api.render_static(ctx, plan, ds, prm, got)
    torch.cuda.synchronize()
    assert torch.equal(got, ref) and float(ref.sum()) > 0
