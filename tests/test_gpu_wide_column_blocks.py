"""Completion in global memory and masked ALS with column blocks of 256: a rank bucket of at least 2,048 such blocks
takes them, fewer take blocks of 64 columns (which every plan of one slice does).  Slices of 255 to 515 columns: a
block short of a column, full, one column over, three blocks; a column of every row, an empty one.  Against the FP64
oracle on the same samples, for slices of each shape at both ends of the bucket.  1e-3 per slice: the per-slice bar of
every completion test, three orders above the FP32 rounding of the Grams."""
import types

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import render as orender  # noqa: E402
from oracle.sampling import count_from_ppm  # noqa: E402
from paper_2202_12567_amd import api  # noqa: E402

SEED = 4
PPM = 200000
SHAPES = [(40, 257), (300, 255), (33, 256), (48, 300), (35, 515), (200, 258)]


def samples_of(m, n, rng):
    N1 = count_from_ppm(PPM, m * n)
    first = np.arange(m) * n + n // 2                        # a column of every row
    rest = rng.permutation(m * n)[:N1 + 2 * m]
    rest = rest[(rest % n != n // 2) & (rest % n != n - 1)]  # the last column stays empty
    e = np.concatenate([first, rest])[:N1]
    assert e.shape[0] == N1
    return rng.permutation(e)


@pytest.mark.parametrize("method,q", [("adm", 20), ("adm", 32), ("als", 4), ("als", 16), ("als", 32)])
def test_wide_column_blocks(method, q):
    iters = 5 if method == "adm" else 3
    shapes = []
    while sum((n + 255) // 256 for _, n in shapes) < 2048:
        shapes.append(SHAPES[len(shapes) % len(SHAPES)])
    m, n = (np.array([s[k] for s in shapes]) for k in (0, 1))
    off = np.concatenate([[0], np.cumsum(m)]).astype(np.int32)
    lay = types.SimpleNamespace(n_slices=len(shapes), n_clusters=int(n.max()), pt_offsets=off,
                                cl_offsets=np.concatenate([[0], np.cumsum(n)]).astype(np.int32),
                                rank=np.full(len(shapes), q, np.int32))
    prm = api.default_params(seed=SEED, pass1_ppm=PPM, pass2_ppm=0, max_iter=iters, fixed_iters=True, als=method == "als")
    dev = torch.device("cuda", 0)
    ctx, plan = api.Context(0), api.Plan(lay, prm)
    assert not plan.slice_info(0)["adm_in_lds"]
    ws = api.workspace(plan, dev)
    rng = np.random.default_rng(q)
    # one pattern of samples per shape, values of their own for every slice
    pattern = [samples_of(a, b, rng) for a, b in SHAPES]
    keys = [((e // b) << 16 | e % b).astype(np.int32) for e, (a, b) in zip(pattern, SHAPES)]
    keys = np.concatenate([keys[s % len(SHAPES)] for s in range(len(shapes))])
    vals = rng.uniform(0.1, 2.0, (keys.shape[0], 3)).astype(np.float32)
    api.region_view(plan, ws, "OMEGA1", torch.int32)[:keys.shape[0]] = torch.as_tensor(keys, device=dev)
    api.region_view(plan, ws, "VAL1", torch.float32)[:vals.size] = torch.as_tensor(vals.ravel(), device=dev)
    pt = torch.arange(int(off[-1]), dtype=torch.int32, device=dev)
    rad = api.stage_adm(ctx, plan, prm, pt, ws, n_points=int(off[-1])).double().cpu().numpy()
    st = api.read_stats(ctx, plan, ws)
    at = np.concatenate([[0], np.cumsum([pattern[s % len(SHAPES)].shape[0] for s in range(len(shapes))])])
    ends = list(range(len(SHAPES))) + list(range(len(shapes) - len(SHAPES), len(shapes)))
    for s in ends:
        e = pattern[s % len(SHAPES)]
        want, n_it, err, _, _ = orender.complete_and_render(
            int(m[s]), int(n[s]), q, e // n[s], e % n[s], vals[at[s]:at[s + 1]].astype(np.float64), SEED, s,
            orender.Params(seed=SEED, max_iter=iters, fixed_iters=True, method=method, lam=0.01))
        assert int(st["iters"][s]) == n_it == iters
        assert abs(float(st["resid"][s]) - err) <= 1e-3 * err + 1e-6, s
        assert orender.relative_rmse(rad[off[s]:off[s + 1]], want) <= 1e-3, s
