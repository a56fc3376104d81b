"""The split test's two forms (levels of few nodes, a workgroup per node; levels of many, nodes in groups) at the sample
counts where a thread takes 1, 2 or 4 samples (256, 512) and a tree deep enough for both, against the FP64 oracle at the
light cut's bounds (seed 34: the oracle has no decision within its tie margin at any of these counts); and sample pixels
given twice leave every node's largest ratio as it was, bit for bit, at counts on either side of those lines."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import lightcut as LC  # noqa: E402
from test_gpu_lightcut import ctx, compare, gpu_cut  # noqa: E402,F401
from test_oracle_lightcut import _random_frame, _scene  # noqa: E402


@pytest.mark.parametrize("S", [255, 256, 257, 511, 512, 513])
@pytest.mark.parametrize("nv", [2, 700, 5000])
def test_samples_per_thread(ctx, nv, S):  # noqa: F811
    pts, vp, perm, left, right = _random_frame(34 + nv, nv=nv, m=S)
    o = LC.lightcut(pts, vp, perm, left, right, np.arange(S), 0.01, 10_000, seed=34)
    g = gpu_cut(ctx, _scene(pts, vp), perm, left, right, np.arange(S), 0.01, 10_000, seed=34)
    compare(g, o)


@pytest.mark.parametrize("S", [200, 400, 900])
def test_samples_twice(ctx, S):  # noqa: F811
    pts, vp, perm, left, right = _random_frame(37, nv=5000, m=S)
    sc = _scene(pts, vp)
    a, b = (gpu_cut(ctx, sc, perm, left, right, np.tile(np.arange(S), k), 0.01, 10_000, seed=37) for k in (1, 2))
    for k in a:
        assert np.array_equal(a[k], b[k]), k
