"""Masked ALS with the residual stop, and what its runs may not depend on: the order in which workgroups are done,
values that no sample reads, and the iteration limit once every slice has stopped."""
import time
import types

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import render as orender  # noqa: E402
from paper_2202_12567_amd import api  # noqa: E402

DEV = torch.device("cuda", 0)
SEED = 9
PPM = 400000


class Workload:
    """Slices (m, n, q, noise): a positive matrix of two components per channel and relative noise, 40% sampled."""

    def __init__(self, slices, seed=1, holes=False, **prm):
        rng = np.random.default_rng(seed)
        m, n, q = (np.array([s[k] for s in slices], np.int64) for k in range(3))
        off = np.concatenate([[0], np.cumsum(m)]).astype(np.int32)
        lay = types.SimpleNamespace(n_slices=len(slices), n_clusters=int(n.max()), pt_offsets=off,
                                    cl_offsets=np.concatenate([[0], np.cumsum(n)]).astype(np.int32),
                                    rank=q.astype(np.int32))
        self.prm = api.default_params(seed=SEED, pass1_ppm=PPM, pass2_ppm=0, als=True, **prm)
        self.ctx, self.plan = api.Context(0), api.Plan(lay, self.prm)
        self.rows, self.slices, self.samples = int(off[-1]), slices, []
        keys, vals = [], []
        for ms, ns, _, noise in slices:
            N1 = (PPM * ms * ns + 500000) // 1000000
            e = rng.permutation((ms - 1 if holes else ms) * ns)[:N1]      # holes: no sample in the last row
            assert e.shape[0] == N1
            M = (rng.uniform(0.1, 1, (ms, 2)) @ rng.uniform(0.1, 1, (2, 3 * ns))).reshape(ms, ns, 3)
            v = (M[e // ns, e % ns] * rng.uniform(1 - noise, 1 + noise, (N1, 3))).astype(np.float32)
            keys.append((e // ns << 16 | e % ns).astype(np.int32))
            vals.append(v)
            self.samples.append((e // ns, e % ns, v))
        self.keys = torch.as_tensor(np.concatenate(keys), device=DEV)
        self.vals = torch.as_tensor(np.concatenate(vals).ravel(), device=DEV)
        self.pt = torch.arange(self.rows, dtype=torch.int32, device=DEV)

    def workspace(self):
        ws = api.workspace(self.plan, DEV).zero_()
        api.region_view(self.plan, ws, "OMEGA1", torch.int32)[:self.keys.shape[0]] = self.keys
        api.region_view(self.plan, ws, "VAL1", torch.float32)[:self.vals.shape[0]] = self.vals
        return ws

    def run(self, ws):
        return api.stage_adm(self.ctx, self.plan, self.prm, self.pt, ws, n_points=self.rows)

    def stats(self, ws):
        return api.read_stats(self.ctx, self.plan, ws)

    def x(self, ws):
        return api.region_view(self.plan, ws, "X", torch.float32).clone()


def test_whole_workspace_repeats():
    """Thousands of rows with equal sample counts: every byte a run leaves behind is the same."""
    w = Workload([(900, 40, 8, 0.05)] * 6 + [(500, 300, 16, 0.05)] * 6, max_iter=6, tol=1e-9)
    first = w.workspace()
    w.run(first)
    for _ in range(6):
        ws = w.workspace()
        w.run(ws)
        assert torch.equal(ws, first)


@pytest.mark.parametrize("m,n,q", [(33, 20, 4), (150, 90, 16)])
def test_given_factors_of_a_row_without_samples_are_not_read(m, n, q):
    """Nor are they by the oracle: the residual is over the samples."""
    res = []
    for fill in (0.25, float("nan"), float("inf")):
        w = Workload([(m, n, q, 0.02)], holes=True, given_init=True, max_iter=1, tol=1e-9)
        ws = w.workspace()
        g = torch.Generator().manual_seed(3)
        for name, count in (("X", m * q), ("Y", 3 * n * q)):
            api.region_view(w.plan, ws, name, torch.float32)[:count] = torch.rand(count, generator=g).to(DEV)
        api.region_view(w.plan, ws, "X", torch.float32)[(m - 1) * q:m * q] = fill
        rad = w.run(ws)
        res.append((float(w.stats(ws)["resid"][0]), rad))
    for resid, rad in res:
        assert np.isfinite(resid) and resid == res[0][0] and torch.equal(rad, res[0][1])


SMALL = [(64, 64, 8, 0.02), (40, 30, 4, 0.3), (50, 64, 16, 0.1), (33, 17, 3, 0.15), (64, 20, 12, 0.25)]
LARGE = [(200, 70, 8, 0.02), (130, 300, 16, 0.25), (70, 260, 4, 0.3), (300, 40, 12, 0.15), (90, 100, 32, 0.1)]


@pytest.mark.parametrize("slices,tol,iters", [(SMALL, 0.08, [2, 8, 1, 3, 2]), (LARGE, 0.11, [1, 3, 8, 2, 1])])
def test_stops_where_the_oracle_does(slices, tol, iters):
    """Slices that stop after odd, even and no iterations (the oracle's residuals before and after a stop are at least
    2% off the tolerance; FP32 Grams move them by 1e-5), the launches' tiles of rows and columns crossed."""
    w = Workload(slices, max_iter=8, tol=tol)
    ws = w.workspace()
    rad = w.run(ws).double().cpu().numpy()
    st, at = w.stats(ws), 0
    assert [int(k) for k in st["iters"]] == iters
    for s, (m, n, q, _) in enumerate(slices):
        ii, jj, v = w.samples[s]
        want, n_it, err, flags, _ = orender.complete_and_render(
            m, n, q, ii, jj, v.astype(np.float64), SEED, s,
            orender.Params(seed=SEED, max_iter=8, fixed_iters=False, tol=tol, method="als", lam=0.01))
        assert n_it == iters[s]
        assert abs(float(st["resid"][s]) - err) <= 1e-3 * err
        assert bool(int(st["flags"][s]) & 2) == (n_it == 8)
        assert orender.relative_rmse(rad[at:at + m], want) <= 1e-3
        at += m


@pytest.mark.parametrize("slices", [SMALL, LARGE])
@pytest.mark.parametrize("iters", [5, 131, 160])
def test_an_unreached_tolerance_gives_the_factors_of_the_fixed_count(slices, iters):
    """Bit for bit, past the iterations that are launches of their own too."""
    got = []
    for prm in (dict(tol=1e-12), dict(fixed_iters=True)):
        w = Workload(slices, max_iter=iters, **prm)
        ws = w.workspace()
        rad = w.run(ws)
        assert [int(k) for k in w.stats(ws)["iters"]] == [iters] * len(slices)
        got.append((rad, w.x(ws)))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("slices", [SMALL, LARGE])
def test_a_high_limit_costs_little_once_every_slice_has_stopped(slices):
    """Every slice stops before its third iteration; the limit of 3,000 takes no more than five times that of 100 (an
    empty launch per half-step took thirty times)."""
    took = []
    for limit in (100, 3000):
        w = Workload(slices, max_iter=limit, tol=0.3)
        ws = w.workspace()
        times = []
        for _ in range(7):
            torch.cuda.synchronize()
            t = time.perf_counter()
            w.run(ws)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t)
        assert max(int(k) for k in w.stats(ws)["iters"]) < 3
        took.append(sorted(times)[3])
    assert took[1] <= 5 * took[0]
