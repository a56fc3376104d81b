"""The work this library is used for, as timed cases.

A case is a dict of plain values; its "kind" is one of

  frame      a whole frame through ``api.render``: cluster table, (light
             coarsening,) both sampling passes, entries with shadow rays,
             completion, factorised sum; returns the radiance
  complete   the completion of caller samples through ``api.stage_adm``
             (non-negative ADM, or masked ALS); returns the radiance and the
             slice scales
  entries    lighting-matrix entries of (point, light) pairs through
             ``api.eval_pairs``
  reference  the brute-force column sum of reference images
             (``api.brute_force``)
  light_cut  the global light cut of a whole light tree (``api.lightcut``)
  train      one training step of the proposal network
             (``api.mlp_train_step``); returns the updated parameters, both
             moments and the loss

Scenes follow the recipe of the repository's workloads (spheres, or icosphere
meshes, resting on a plane under an orthographic camera; VPLs above them; a
median-split light tree; slices by bisection of position and normal), drawn on
the GPU so that a fresh scene takes well under a second.
"""
import math
import os
from types import SimpleNamespace

import numpy as np
import torch

import paper_2202_12567_amd as package
from paper_2202_12567_amd import api

DEV = torch.device("cuda", 0)
F32, F64 = torch.float32, torch.float64

# Entries of one shading evaluation cost about 60 FLOP, a traversed BVH node
# about 20; a shadow ray meets some 20 nodes of these scenes.
ENTRY_FLOPS = 60.0
RAY_FLOPS = 400.0
POINT_BYTES, LIGHT_BYTES = 44.0, 36.0


def listed():
    return [
        # smallest frame, the tests' and the smoke run's: a preview of 64x64
        # points under 1,024 single VPLs
        {"name": "frame_tiny", "kind": "frame", "width": 64, "height": 64, "spheres": 32, "mesh": False,
         "vpls": 1024, "clusters": 1024, "phong": 0.0, "slices": 16, "slice_max": 0, "rank": 8, "ppm1": 50000,
         "ppm2": 50000, "draws": 0, "n_max": 0, "learned": False},
        # an ordinary frame without coarsening: 512x512 points, 65,536 VPLs
        # cut to 4,096 clusters, 5% of every slice sampled
        {"name": "frame_mid", "kind": "frame", "width": 512, "height": 512, "spheres": 512, "mesh": False,
         "vpls": 65536, "clusters": 4096, "phong": 0.5, "slices": 256, "slice_max": 0, "rank": 16, "ppm1": 25000,
         "ppm2": 25000, "draws": 0, "n_max": 0, "learned": False},
        # the benchmark's frame and the largest case: 1920x1080, 300,000
        # VPLs, every slice coarsened from 16,384 clusters to 512 columns
        {"name": "frame_hd", "kind": "frame", "width": 1920, "height": 1080, "spheres": 2048, "mesh": False,
         "vpls": 300000, "clusters": 16384, "phong": 1.0, "slices": 0, "slice_max": 1024, "rank": 16, "ppm1": 0,
         "ppm2": 10000, "draws": 32768, "n_max": 512, "learned": False},
        # a triangle scene with VPLs on its surfaces, its second pass drawn
        # by the learned proposal
        {"name": "frame_tri_learned", "kind": "frame", "width": 256, "height": 256, "spheres": 128, "mesh": True,
         "vpls": 16384, "clusters": 2048, "phong": 0.5, "slices": 64, "slice_max": 0, "rank": 16, "ppm1": 25000,
         "ppm2": 25000, "draws": 0, "n_max": 0, "learned": True},
        # completion alone, slices as a coarsened frame has them (uneven
        # rows, 512 columns, a few percent sampled with skewed columns)
        {"name": "complete_rank16", "kind": "complete", "slices": 256, "rows_min": 50, "rows_max": 1024, "cols": 512,
         "rank": 16, "ppm": 65000, "method": "adm"},
        # the same at the highest rank, whose factors exceed LDS
        {"name": "complete_rank32", "kind": "complete", "slices": 96, "rows_min": 300, "rows_max": 1024, "cols": 512,
         "rank": 32, "ppm": 65000, "method": "adm"},
        # masked ALS, the more accurate completion variant
        {"name": "complete_als", "kind": "complete", "slices": 48, "rows_min": 200, "rows_max": 900, "cols": 300,
         "rank": 16, "ppm": 65000, "method": "als"},
        # a handful of entries (a probe under the cursor): latency
        {"name": "entries_probe", "kind": "entries", "pairs": 3001, "points": 4096, "lights": 1024, "spheres": 32,
         "mesh": False, "phong": 0.5},
        # many entries of a triangle scene
        {"name": "entries_tri", "kind": "entries", "pairs": 2000000, "points": 65536, "lights": 16384, "spheres": 128,
         "mesh": True, "phong": 0.5},
        # reference pixels against every light
        {"name": "reference", "kind": "reference", "pixels": 8192, "points": 262144, "lights": 16384, "spheres": 512,
         "phong": 0.5},
        # step 1 of the method at 1080p: the cut of 300,000 VPLs
        {"name": "light_cut", "kind": "light_cut", "vpls": 300000, "samples": 8192, "points": 262144, "spheres": 512,
         "phong": 1.0, "eps": 0.02, "max_cut": 16384},
        # one step of the proposal's training (128 slices of 1,024 columns)
        {"name": "train_step", "kind": "train", "groups": 128, "group_rows": 1024},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame", "frame", "coarse", "complete", "complete", "als", "entries", "reference", "light_cut",
                       "train"])
    if kind == "frame":
        side = _log(rng, 64, 520)
        return {"kind": "frame", "width": side + rng.randrange(8), "height": side, "spheres": _log(rng, 16, 512),
                "mesh": False, "vpls": _log(rng, 4096, 65536), "clusters": _log(rng, 256, 4096),
                "phong": rng.choice([0.0, 0.5, 1.0]), "slices": 0, "slice_max": rng.choice([256, 700, 1024, 1500]),
                "rank": rng.choice([4, 7, 8, 12, 16, 32]), "ppm1": rng.randrange(5000, 50000),
                "ppm2": rng.randrange(2500, 50000), "draws": 0, "n_max": 0, "learned": rng.random() < 0.3}
    if kind == "coarse":
        side = _log(rng, 128, 900)
        return {"kind": "frame", "width": side + rng.randrange(8), "height": side, "spheres": _log(rng, 64, 2048),
                "mesh": False, "vpls": _log(rng, 16384, 200000), "clusters": _log(rng, 1024, 16384),
                "phong": rng.choice([0.5, 1.0]), "slices": 0, "slice_max": rng.choice([512, 1024]),
                "rank": rng.choice([8, 16, 32]), "ppm1": 0, "ppm2": rng.randrange(5000, 50000),
                "draws": _log(rng, 8192, 32768), "n_max": _log(rng, 200, 700), "learned": False}
    if kind == "complete":
        rank = rng.choice([5, 8, 16, 16, 24, 32])
        return {"kind": "complete", "slices": _log(rng, 16, 200), "rows_min": _log(rng, 40, 300),
                "rows_max": _log(rng, 310, 2000 if rank < 16 else 1100), "cols": _log(rng, 128, 1500), "rank": rank,
                "ppm": rng.randrange(20000, 90000), "method": "adm"}
    if kind == "als":
        return {"kind": "complete", "slices": _log(rng, 8, 48), "rows_min": _log(rng, 40, 200),
                "rows_max": _log(rng, 210, 900), "cols": _log(rng, 64, 512), "rank": rng.choice([8, 12, 16]),
                "ppm": rng.randrange(20000, 90000), "method": "als"}
    if kind == "entries":
        return {"kind": "entries", "pairs": _log(rng, 1000, 4000000), "points": _log(rng, 4096, 262144),
                "lights": _log(rng, 500, 65536), "spheres": _log(rng, 16, 1024), "mesh": False,
                "phong": rng.choice([0.0, 0.5, 1.0])}
    if kind == "reference":
        return {"kind": "reference", "pixels": _log(rng, 64, 8192), "points": _log(rng, 16384, 262144),
                "lights": _log(rng, 1000, 16384), "spheres": _log(rng, 16, 1024), "phong": rng.choice([0.0, 0.5, 1.0])}
    if kind == "light_cut":
        return {"kind": "light_cut", "vpls": _log(rng, 4096, 300000), "samples": _log(rng, 256, 8192),
                "points": _log(rng, 16384, 262144), "spheres": _log(rng, 32, 512), "phong": rng.choice([0.0, 0.5, 1.0]),
                "eps": rng.choice([0.01, 0.02, 0.05]), "max_cut": _log(rng, 512, 16384)}
    return {"kind": "train", "groups": _log(rng, 8, 160), "group_rows": _log(rng, 100, 1100)}


# ---------------------------------------------------------------------------
# scenes
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _u(g, lo, hi, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=F64) * (hi - lo) + lo


def _icosphere(level):
    """Unit icosphere faces (F, 3, 3), wound outwards."""
    t = (1.0 + math.sqrt(5.0)) / 2.0
    v = [np.array(p, float) for p in ((0, 1, t), (0, -1, t), (0, 1, -t), (0, -1, -t), (1, t, 0), (-1, t, 0), (1, -t, 0),
                                      (-1, -t, 0), (t, 0, 1), (t, 0, -1), (-t, 0, 1), (-t, 0, -1))]
    v = np.stack([p / np.linalg.norm(p) for p in v])
    edge = min(np.linalg.norm(v[0] - p) for p in v[1:]) * 1.01
    near = np.linalg.norm(v[:, None] - v[None], axis=2) < edge
    f = np.array([(v[a], v[b], v[c]) for a in range(12) for b in range(a + 1, 12) for c in range(b + 1, 12)
                  if near[a, b] and near[b, c] and near[a, c]])
    for _ in range(level):
        a, b, c = f[:, 0], f[:, 1], f[:, 2]
        ab, bc, ca = (p / np.linalg.norm(p, axis=1, keepdims=True) for p in (a + b, b + c, c + a))
        f = np.concatenate([np.stack(q, 1) for q in ((a, ab, ca), (ab, b, bc), (ca, bc, c), (ab, bc, ca))])
    flip = np.einsum("fk,fk->f", np.cross(f[:, 1] - f[:, 0], f[:, 2] - f[:, 0]), f.mean(1)) < 0
    f[flip] = f[flip][:, [0, 2, 1]]
    return torch.as_tensor(f, device=DEV)


def _first_hit(o, d, sph, faces):
    """Nearest hit of rays on the plane z = 0 and the icospheres: position, normal, object."""
    t = -o[:, 2] / d[:, 2]
    n = torch.zeros_like(o)
    n[:, 2] = 1.0
    obj = torch.zeros(o.shape[0], dtype=torch.int64, device=DEV)
    for k in range(sph.shape[0]):
        c, r = sph[k, :3], sph[k, 3]
        oc = c - o
        tc = (oc * d).sum(1)
        rows = torch.nonzero((oc * oc).sum(1) - tc * tc <= r * r)[:, 0]
        if rows.numel() == 0:
            continue
        tri = faces * r + c
        e1, e2 = tri[:, 1] - tri[:, 0], tri[:, 2] - tri[:, 0]
        D = d[rows][:, None].expand(-1, tri.shape[0], -1)
        p = torch.linalg.cross(D, e2[None].expand_as(D))
        det = (p * e1).sum(2)
        s = o[rows][:, None] - tri[None, :, 0]
        q = torch.linalg.cross(s, e1[None].expand_as(s))
        u, v, th = (s * p).sum(2) / det, (D * q).sum(2) / det, (q * e2).sum(2) / det
        th = torch.where((u >= 0) & (v >= 0) & (u + v <= 1) & (th > 1e-9), th, math.inf)
        best, f = th.min(1)
        closer = best < t[rows]
        rows, f, best = rows[closer], f[closer], best[closer]
        t[rows] = best
        fn = torch.linalg.cross(e1, e2)
        n[rows] = (fn / fn.norm(dim=1, keepdim=True))[f]
        obj[rows] = k + 1
    return o + t[:, None] * d, n, obj


def _surface(g, width, height, n_spheres, mesh, phong):
    """Points seen by the camera, their materials, and the occluders."""
    region = max(1.0, round(width / height, 3))
    r = _u(g, 0.02, 0.1, n_spheres)
    cx, cy = _u(g, 0.0, region, n_spheres), _u(g, 0.0, 1.0, n_spheres)
    m = width * height
    pix = torch.arange(m, device=DEV)
    X = ((pix % width).double() + 0.5) * (region / width)
    Y = (torch.div(pix, width, rounding_mode="floor").double() + 0.5) / height
    sph = torch.stack([cx, cy, r, r], 1)
    faces = _icosphere(2) if mesh else None
    if mesh:
        o = torch.stack([X, Y, torch.full_like(X, 10.0)], 1)
        d = torch.zeros_like(o)
        d[:, 2] = -1.0
        pos, nrm, obj = _first_hit(o, d, sph, faces)
    else:
        Z = torch.zeros_like(X)
        obj = torch.zeros_like(pix)
        for k in range(0, n_spheres, 32):
            d2 = (X[None] - cx[k:k + 32, None]) ** 2 + (Y[None] - cy[k:k + 32, None]) ** 2
            h = r[k:k + 32, None] ** 2 - d2
            z = torch.where(h > 0, r[k:k + 32, None] + torch.sqrt(h.clamp(min=0)), -1.0)
            zb, kb = z.max(0)
            hit = zb > Z
            Z = torch.where(hit, zb, Z)
            obj = torch.where(hit, kb + (k + 1), obj)
        pos = torch.stack([X, Y, Z], 1)
        c = torch.cat([torch.zeros(1, 4, device=DEV, dtype=F64), sph])[obj]
        nrm = torch.where((obj > 0)[:, None], pos - c[:, :3], torch.tensor([0.0, 0.0, 1.0], device=DEV, dtype=F64))
        nrm = nrm / nrm.norm(dim=1, keepdim=True)
    albedo = _u(g, 0.2, 0.9, n_spheres + 1, 3)
    shiny = _u(g, 0.0, 1.0, n_spheres + 1) < phong
    expo = torch.where(shiny, _u(g, 10.0, 100.0, n_spheres + 1), 1.0)
    kd = torch.where(shiny[:, None], 0.75 * albedo, albedo)
    ks = torch.where(shiny, 0.2, 0.0)
    pts = torch.cat([pos, nrm, kd[obj], ks[obj, None], expo[obj, None]], 1).to(F32)
    if mesh:
        tri = (sph[:, None, None, :3] + r[:, None, None, None] * faces[None]).reshape(-1, 9)
        a, b = -1.0, region + 1.0
        ground = torch.tensor([[a, -1, 0, b, -1, 0, b, 2, 0], [a, -1, 0, b, 2, 0, a, 2, 0]], device=DEV, dtype=F64)
        occ = {"tri": torch.cat([ground, tri]).to(F32).cpu().numpy()}
    else:
        occ = {k: v.to(F32).cpu().numpy() for k, v in zip(("cx", "cy", "cz", "r"), (cx, cy, r, r))}
    return pts, occ, region, (sph, faces, kd)


def _lights(g, n, region, mesh_of=None):
    """VPLs above the scene, or (meshes) the first bounces of paths from a disk light: (n, 9) position, normal, RGB."""
    if mesh_of is None:
        pos = torch.stack([_u(g, 0.0, region, n), _u(g, 0.0, 1.0, n), _u(g, 0.25, 1.0, n)], 1)
        rr, ph = _u(g, 0.0, 1.0, n), _u(g, 0.0, 2 * math.pi, n)
        d = torch.stack([rr.sqrt() * ph.cos(), rr.sqrt() * ph.sin(), (1 - rr).clamp(min=0).sqrt()], 1)
        return torch.cat([pos, -d / d.norm(dim=1, keepdim=True), _u(g, 0.0, 1.0, n, 3)], 1).to(F32)
    sph, faces, kd = mesh_of
    got = []
    while sum(x.shape[0] for x in got) < n:
        k = 2 * n + 64
        rad, ph = 0.3 * _u(g, 0.0, 1.0, k).sqrt(), _u(g, 0.0, 2 * math.pi, k)
        o = torch.stack([0.5 * region + rad * ph.cos(), 0.5 + rad * ph.sin(), torch.full_like(rad, 2.0)], 1)
        u1, ph = _u(g, 0.0, 0.98, k), _u(g, 0.0, 2 * math.pi, k)
        d = torch.stack([u1.sqrt() * ph.cos(), u1.sqrt() * ph.sin(), -(1 - u1).sqrt()], 1)
        p, nrm, obj = _first_hit(o, d, sph, faces)
        ok = (p[:, 0] >= 0) & (p[:, 0] <= region) & (p[:, 1] >= 0) & (p[:, 1] <= 1)
        got.append(torch.cat([p + 2e-3 * nrm, nrm, kd[obj] * (1000.0 / n)], 1)[ok])
    return torch.cat(got)[:n].to(F32)


def _split_sizes(n, leaves):
    """Level by level the (start, size, leaves) of a tree over n items grown to `leaves` leaves by halving."""
    levels = [(np.array([0]), np.array([n]), np.array([leaves]))]
    while (levels[-1][2] > 1).any():
        st, sz, lv = levels[-1]
        big = lv > 1
        la = np.where(big, lv // 2, lv)
        sa = np.where(big, np.maximum(la, np.minimum(sz - (lv - la), np.round(sz * (la / lv)).astype(np.int64))), sz)
        st2, sz2, lv2 = (np.stack(p, 1) for p in ((st, st + sa), (sa, sz - sa), (la, lv - la)))
        keep = np.stack([np.ones_like(big), big], 1)
        levels.append((st2[keep], sz2[keep], lv2[keep]))
    return levels


def _light_tree(pos, leaves):
    """Median-split light tree over the rows of pos, `leaves` leaves.  Returns the items ordered by leaf (leaves in tree
    order), the leaves' sizes, and the children of the split nodes: leaf x is node x, split nodes follow, deepest first,
    the root last."""
    n = pos.shape[0]
    perm = torch.arange(n, device=DEV)
    levels = _split_sizes(n, leaves)
    for st, sz, lv in levels[:-1]:
        seg = torch.repeat_interleave(torch.arange(len(sz), device=DEV), torch.as_tensor(sz, device=DEV))
        p = pos[perm]
        ext = torch.stack([torch.full((len(sz), 3), s * 1e9, device=DEV, dtype=p.dtype).scatter_reduce(
            0, seg[:, None].expand(-1, 3), p, how) for s, how in ((1, "amin"), (-1, "amax"))])
        axis = (ext[1] - ext[0]).argmax(1)
        key = p.gather(1, axis[seg][:, None])[:, 0]
        key = torch.where(torch.as_tensor(lv > 1, device=DEV)[seg], key, torch.zeros_like(key))
        o = torch.sort(key, stable=True)[1]
        perm = perm[o[torch.sort(seg[o], stable=True)[1]]]
    # node ids: leaves in order, split nodes from the deepest level up
    ids, left, right, nid = np.arange(leaves), [], [], leaves
    for st, sz, lv in reversed(levels[:-1]):
        up, k = np.empty(len(lv), np.int64), 0
        for i, v in enumerate(lv):
            if v > 1:
                left.append(ids[k])
                right.append(ids[k + 1])
                up[i] = nid
                nid, k = nid + 1, k + 2
            else:
                up[i] = ids[k]
                k += 1
        ids = up
    return perm, levels[-1][1], np.array(left, np.int32), np.array(right, np.int32)


def _slices(pts, count, biggest):
    """Point ids slice by slice and the slices' sizes: `count` equal slices (a power of two), or bisection at the
    midpoint down to at most `biggest` points."""
    pos, nrm = pts[:, :3].double(), pts[:, 3:6].double()
    feat = torch.cat([pos / (pos.amax(0) - pos.amin(0)).norm(), 0.5 * nrm], 1)
    ids = torch.arange(pts.shape[0], device=DEV)
    seg = torch.zeros_like(ids)
    level = 0
    while True:
        n_seg = int(seg.max()) + 1
        size = torch.bincount(seg, minlength=n_seg)
        if (1 << level) >= count if count else int(size.max()) <= biggest:
            return ids, size.cpu().numpy()
        f = feat[ids]
        lo, hi = (torch.full((n_seg, 6), s * 1e9, device=DEV, dtype=F64).scatter_reduce(
            0, seg[:, None].expand(-1, 6), f, how) for s, how in ((1, "amin"), (-1, "amax")))
        axis = (hi - lo).argmax(1)
        x = f.gather(1, axis[seg][:, None])[:, 0]
        first = torch.cumsum(size, 0) - size
        if count:
            o = torch.sort(x, stable=True)[1]
            o = o[torch.sort(seg[o], stable=True)[1]]
            ids, seg = ids[o], seg[o]
            side = (torch.arange(ids.numel(), device=DEV) - first[seg] >= size[seg] // 2).long()
        else:
            mid = 0.5 * (lo + hi).gather(1, axis[:, None])[:, 0]
            side = ((x >= mid[seg]) & (size > biggest)[seg]).long()
        o = torch.sort(2 * seg + side, stable=True)[1]
        ids = ids[o]
        seg = torch.unique_consecutive((2 * seg + side)[o], return_inverse=True)[1]
        level += 1


def _planes(t, keys):
    a = t.t().contiguous().cpu().numpy()
    return {k: a[i] for i, k in enumerate(keys)}


def _frame_scene(case, seed):
    g = _gen(seed)
    pts, occ, region, mesh = _surface(g, case["width"], case["height"], case["spheres"], case["mesh"], case["phong"])
    vpl = _lights(g, case["vpls"], region, mesh if case["mesh"] else None)
    nc = min(case["clusters"], case["vpls"])
    perm, sizes, left, right = _light_tree(vpl[:, :3].double(), nc)
    # clusters in the order of their smallest member, as a cut table lists them
    leaf = np.repeat(np.arange(nc), sizes)
    perm = perm.cpu().numpy()
    small = np.minimum.reduceat(perm, np.concatenate([[0], np.cumsum(sizes)[:-1]]))
    rank_of = np.empty(nc, np.int64)
    rank_of[np.argsort(small)] = np.arange(nc)
    order = np.lexsort((perm, rank_of[leaf]))
    offsets = np.concatenate([[0], np.cumsum(sizes[np.argsort(small)])])
    node = np.concatenate([rank_of, np.arange(nc, 2 * nc - 1)])
    ids, m_s = _slices(pts, case["slices"], case["slice_max"])
    S = len(m_s)
    coarse = case["draws"] > 0
    i32 = lambda a: np.asarray(a, np.int32)  # noqa: E731
    return SimpleNamespace(
        points=_planes(pts, api.DeviceScene.POINT_KEYS), vpls=_planes(vpl, api.DeviceScene.LIGHT_KEYS), spheres=occ,
        cut_offsets=i32(offsets), cut_members=i32(perm[order]), pt_offsets=i32(np.concatenate([[0], np.cumsum(m_s)])),
        pt_ids=i32(ids.cpu().numpy()), cl_offsets=i32(np.arange(S + 1) * nc),
        cl_ids=np.zeros(1, np.int32) if coarse else np.tile(np.arange(nc, dtype=np.int32), S),
        rank=i32(np.minimum(case["rank"], np.minimum(m_s, nc))), tree_left=i32(node[left]), tree_right=i32(node[right]),
        m=pts.shape[0], n=vpl.shape[0], n_clusters=nc, n_slices=S)


def _entry_scene(case, seed):
    """A scene whose lights are used one by one: (context, device scene, occluder spheres, generator)."""
    g = _gen(seed)
    side = max(16, int(math.sqrt(case["points"])))
    mesh = case.get("mesh", False)
    pts, occ, region, geo = _surface(g, side, side, case["spheres"], mesh, case["phong"])
    vpl = _lights(g, case.get("lights", case.get("vpls")), region, geo if mesh else None)
    one = np.zeros(1, np.int32)
    sc = SimpleNamespace(points=_planes(pts, api.DeviceScene.POINT_KEYS), vpls=_planes(vpl, api.DeviceScene.LIGHT_KEYS),
                         spheres=occ, cut_offsets=np.array([0, vpl.shape[0]], np.int32),
                         cut_members=np.arange(vpl.shape[0], dtype=np.int32), pt_ids=one, cl_ids=one, m=pts.shape[0],
                         n=vpl.shape[0], n_clusters=1)
    return sc, pts, vpl, geo, g


# ---------------------------------------------------------------------------
# entries in 64 bits
# ---------------------------------------------------------------------------

R_MIN, RAY_EPS = 0.05, 1e-4


def _shade64(P, L, visible):
    """Entries (k, 3) of point rows P (k, 11) and light rows L (k, 9) in 64 bits."""
    P, L = P.double(), L.double()
    x, n = P[:, :3], P[:, 3:6]
    d = L[:, :3] - x
    r2 = (d * d).sum(1)
    w = d / r2.sqrt()[:, None]
    cx, cy = (n * w).sum(1), -(L[:, 3:6] * w).sum(1)
    lit = (cx > 0) & (cy > 0)
    G = cx * cy / r2.clamp(min=float(np.float32(R_MIN)) ** 2)
    cr = (2 * cx * n[:, 2] - w[:, 2]).clamp(min=0)
    spec = torch.where(P[:, 9] > 0, P[:, 9] * (P[:, 10] + 2) / (2 * math.pi) * cr ** P[:, 10], 0.0)
    f = P[:, 6:9] / math.pi + spec[:, None]
    o = x + float(np.float32(RAY_EPS)) * n
    v = torch.zeros_like(lit)
    v[lit] = visible(o[lit], L[lit, :3] - o[lit])
    return torch.where(v[:, None], f * L[:, 6:9] * G[:, None], 0.0)


def _visible64(geo, occ):
    """Visibility of segments o + t D, t in (0, 1), against spheres or their icospheres on the ground."""
    if "tri" not in occ:
        c = torch.as_tensor(np.stack([occ[k] for k in ("cx", "cy", "cz", "r")], 1), device=DEV).double()

        def spheres(o, D):
            free = torch.ones(o.shape[0], dtype=torch.bool, device=DEV)
            inv = 1.0 / (D * D).sum(1)
            step = max(1, (1 << 25) // max(1, o.shape[0]))
            oD = (o * D).sum(1)
            for k in range(0, c.shape[0], step):
                b = c[k:k + step]
                t = ((D @ b[:, :3].t().contiguous() - oD[:, None]) * inv[:, None]).clamp(0, 1)
                d2 = torch.zeros_like(t)
                for a in range(3):
                    d2 += (b[None, :, a] - o[:, a, None] - t * D[:, a, None]) ** 2
                free &= ~(d2 < b[None, :, 3] ** 2).any(1)
            return free
        return spheres
    tri = torch.as_tensor(occ["tri"], device=DEV).double().reshape(-1, 3, 3)
    parts = [tri[:2]] + list(tri[2:].split((tri.shape[0] - 2) // geo.shape[0]))

    def mesh(o, D):
        free = torch.ones(o.shape[0], dtype=torch.bool, device=DEV)
        for k, T in enumerate(parts):
            rows = torch.nonzero(free)[:, 0]
            if k:
                oc = geo[k - 1, :3] - o[rows]
                t = ((oc * D[rows]).sum(1) / (D[rows] ** 2).sum(1)).clamp(0, 1)
                rows = rows[((oc - t[:, None] * D[rows]) ** 2).sum(1) <= (geo[k - 1, 3] + 1e-5) ** 2]
            e1, e2 = T[:, 1] - T[:, 0], T[:, 2] - T[:, 0]
            for r in rows.split(1 << 16):
                Dr = D[r][:, None].expand(-1, T.shape[0], -1)
                p = torch.linalg.cross(Dr, e2[None].expand_as(Dr))
                det = (p * e1).sum(2)
                s = o[r][:, None] - T[None, :, 0]
                q = torch.linalg.cross(s, e1[None].expand_as(s))
                u, v, t = (s * p).sum(2) / det, (Dr * q).sum(2) / det, (q * e2).sum(2) / det
                hit = (det != 0) & (u >= 0) & (v >= 0) & (u + v <= 1) & (t > 0) & (t < 1)
                free[r[hit.any(1)]] = False
        return free
    return mesh


# ---------------------------------------------------------------------------
# completion: samples and the result in 64 bits
# ---------------------------------------------------------------------------

def _samples(case, seed):
    """Slices of a scene as a coarsened frame has them: rows on a surface patch, skewed column intensities, entries with
    shadows.  Returns rows per slice, sizes, keys, values and row lists."""
    g = _gen(seed)
    S, n, q = case["slices"], case["cols"], case["rank"]
    # log-uniform sizes, the same for every seed, large and small ones mixed
    lo, hi = math.log(case["rows_min"]), math.log(case["rows_max"])
    at = (np.arange(S) * 0.6180339887498949) % 1.0
    m_s = np.maximum(np.round(np.exp(lo + (hi - lo) * at)).astype(np.int64), q)
    n1 = (case["ppm"] * m_s.astype(np.int64) * n + 500000) // 1000000
    sph = torch.cat([_u(g, -0.6, 1.6, 64, 2), _u(g, 0.02, 0.1, 64, 1).repeat(1, 2)], 1)
    keys, vals = [], []
    for s in range(S):
        m = int(m_s[s])
        x = torch.cat([_u(g, 0.0, 0.12, m, 2) + _u(g, 0.0, 0.9, 1, 2), torch.zeros(m, 1, device=DEV, dtype=F64)], 1)
        nr = torch.cat([_u(g, -0.15, 0.15, m, 2) + _u(g, -0.4, 0.4, 1, 2), torch.ones(m, 1, device=DEV, dtype=F64)], 1)
        nr = nr / nr.norm(dim=1, keepdim=True)
        y = torch.stack([_u(g, 0.0, 1.0, n), _u(g, 0.0, 1.0, n), _u(g, 0.25, 1.0, n)], 1)
        weight = torch.exp(0.8 * torch.randn(n, generator=g, device=DEV, dtype=F64))
        inten = weight[:, None] * _u(g, 0.2, 1.0, n, 3)
        # distinct entries, columns in proportion to their intensity
        score = torch.log(_u(g, 1e-12, 1.0, m, n)) / weight
        top = torch.topk(score.reshape(-1), int(n1[s]), sorted=False)[1]
        i, j = torch.div(top, n, rounding_mode="floor"), top % n
        d = y[j] - x[i]
        r2 = (d * d).sum(1)
        cx = (nr[i] * d).sum(1).clamp(min=0) / r2.sqrt()
        G = cx * (d[:, 2] / r2.sqrt()) / r2
        near = sph[((sph[:, :2] - x[0, :2]).norm(dim=1) < 0.6)]
        if near.shape[0]:
            t = ((near[None, :, :3] - x[i][:, None]) * d[:, None]).sum(2) / r2[:, None]
            p = near[None, :, :3] - x[i][:, None] - t.clamp(0, 1)[..., None] * d[:, None]
            G = torch.where(((p * p).sum(2) < near[None, :, 3] ** 2).any(1), 0.0, G)
        keys.append((i << 16 | j).to(torch.int32))
        vals.append((0.3 * G[:, None] * inten[j]).to(F32))
    return m_s, n1, torch.cat(keys), torch.cat(vals)


def _mulhi(a, b):
    """High and low 64 bits of a product of unsigned 64-bit words held as int64."""
    M = 0xFFFFFFFF
    lo = lambda v: v & M  # noqa: E731
    hi = lambda v: (v >> 32) & M  # noqa: E731
    ll, lh, hl = lo(a) * lo(b), lo(a) * hi(b), hi(a) * lo(b)
    mid = hi(ll) + lo(lh) + lo(hl)
    return hi(a) * hi(b) + hi(lh) + hi(hl) + hi(mid), a * b


def _signed(v):
    return v - (1 << 64) if v >> 63 else v


def _philox_u24(k0, k1, c0, c1, tag):
    """Top 24 bits of the first word of Philox4x64-10 (Salmon et al. 2011) as a 32-bit fraction."""
    m0, m1 = (torch.tensor(_signed(v), device=DEV) for v in (0xD2E7470EE14C6C93, 0xCA5A826395121157))
    c0, c1 = torch.broadcast_tensors(c0, c1)
    c2, c3 = torch.full_like(c0, tag), torch.zeros_like(c0)
    for r in range(10):
        a, b = ((k + r * w) & ((1 << 64) - 1) for k, w in ((k0, 0x9E3779B97F4A7C15), (k1, 0xBB67AE8584CAA73B)))
        h0, l0 = _mulhi(c0, m0)
        h1, l1 = _mulhi(c2, m1)
        c0, c1, c2, c3 = h1 ^ c1 ^ _signed(a), l1, h0 ^ c3 ^ _signed(b), l0
    return ((c0 >> 40) & 0xFFFFFF).to(F32) * 2.0 ** -24


def _complete64(case, seed):
    """Radiance of every slice's rows and the scales, in 64 bits (Appendix A in its dense form over padded slices)."""
    m_s, n1, keys, vals = _samples(case, seed)
    S, n, q, M = case["slices"], case["cols"], case["rank"], int(m_s.max())
    prm = _params(case)
    keys, vals = keys.long(), vals.double()
    out, scales = [], []
    start = np.concatenate([[0], np.cumsum(n1)])
    per = max(1, int(4e8 // (M * n * (12 if case["method"] == "adm" else 12 + q * q // 4))))
    for s0 in range(0, S, per):
        ss = range(s0, min(S, s0 + per))
        B = len(ss)
        A = torch.zeros(B, M, 3, n, dtype=F64, device=DEV)
        W = torch.zeros(B, M, n, dtype=F64, device=DEV)
        X, Y = torch.zeros(B, M, q, dtype=F64, device=DEV), torch.zeros(B, q, 3 * n, dtype=F64, device=DEV)
        c = torch.tensor(float(np.float32(2.0 / np.sqrt(float(q)))), device=DEV, dtype=F32)
        mm = torch.as_tensor(m_s[list(ss)], device=DEV).double()[:, None, None]
        scale = []
        for b, s in enumerate(ss):
            k, v = keys[start[s]:start[s + 1]], vals[start[s]:start[s + 1]]
            scale.append(float(v.sum() / (3.0 * v.shape[0])))
            i, j = k >> 16, k & 0xFFFF
            A[b, i, :, j] = v / scale[-1]
            W[b, i, j] = 1.0
            m = int(m_s[s])
            ar = lambda k: torch.arange(k, device=DEV)  # noqa: E731
            X[b, :m] = (_philox_u24(prm.seed, s, ar(m)[:, None], ar(q)[None], 3) * c).double()
            Y[b] = (_philox_u24(prm.seed, s, ar(q)[:, None], ar(3 * n)[None], 4) * c).double()
        A, W3 = A.reshape(B, M, 3 * n), W.repeat(1, 1, 3)
        I = torch.eye(q, dtype=F64, device=DEV)
        T = lambda a: a.transpose(1, 2).contiguous()  # noqa: E731
        f32 = lambda a: float(np.float32(a))  # noqa: E731
        if case["method"] == "adm":
            al, be = f32(prm.alpha0) * 3.0 * n / q, f32(prm.beta0) * mm / q
            ga = f32(prm.gamma)
            U, V, La, Pi = X.clone(), Y.clone(), torch.zeros_like(X), torch.zeros_like(Y)
            for _ in range(prm.max_iter):
                R = W3 * (A - X @ Y)
                Yt = T(Y)
                Gy = Y @ Yt
                Xn = torch.linalg.solve(Gy + al * I, T(X @ Gy + R @ Yt + al * U - La))
                Xn = T(Xn)
                Xt = T(Xn)
                Y2 = torch.linalg.solve(Xt @ Xn + be * I, (Xt @ X) @ Y + Xt @ R + be * V - Pi)
                X, Y = Xn, Y2
                U, V = (X + La / al).clamp(min=0), (Y + Pi / be).clamp(min=0)
                La, Pi = La + ga * al * (X - U), Pi + ga * be * (Y - V)
        else:
            lam = f32(prm.lam)
            for _ in range(prm.max_iter):
                y = T(Y).reshape(B, 3, n, q)
                G = W @ (y[..., :, None] * y[..., None, :]).sum(1).reshape(B, n, q * q)
                cnt = 3.0 * W.sum(2)
                X = torch.linalg.solve(G.reshape(B, M, q, q) + lam * cnt.clamp(min=1)[..., None, None] * I,
                                       ((W3 * A) @ T(Y))[..., None])[..., 0]
                G = T(W) @ (X[..., :, None] * X[..., None, :]).reshape(B, M, q * q)
                cnt = W.sum(1)
                rhs = (T(W3 * A) @ X).reshape(B, 3, n, q).permute(0, 2, 3, 1).contiguous()
                y = torch.linalg.solve(G.reshape(B, n, q, q) + lam * cnt.clamp(min=1)[..., None, None] * I, rhs)
                Y = y.permute(0, 2, 3, 1).reshape(B, q, 3 * n).contiguous()
        Ye = Y.reshape(B, q, 3, n).sum(3)
        I3 = X @ Ye
        for b, s in enumerate(ss):
            out.append(I3[b, :int(m_s[s])] * scale[b])
            scales.append(scale[b])
    return {"radiance": torch.cat(out), "scale": torch.tensor(scales, dtype=F64, device=DEV)}


def _params(case):
    return api.default_params(seed=7, pass1_ppm=case["ppm"], pass2_ppm=0, als=case["method"] == "als")


# ---------------------------------------------------------------------------
# training
# ---------------------------------------------------------------------------

HID, FIN = 128, 12
STEP = 101   # a training under way: 100 steps behind it


def _train_inputs(case, seed):
    """Features, targets, groups, and a network with its moments after some steps."""
    g = _gen(seed)
    rows = case["groups"] * case["group_rows"]
    F = torch.cat([_u(g, 0.0, 3.0, rows, 3), _u(g, 0.0, 2.0, rows, 1), _u(g, 0.0, 1.0, rows, 1),
                   _u(g, 0.0, 1.5, rows, 2), _u(g, -1.0, 1.0, rows, 2), _u(g, 0.0, 2.0, rows, 2),
                   _u(g, 0.0, 0.5, rows, 1)], 1).to(F32)
    sigma = torch.exp(torch.randn(case["groups"], case["group_rows"], generator=g, device=DEV, dtype=F64))
    p = sigma + 3.0 * sigma.mean(1, keepdim=True)
    p = (p / p.sum(1, keepdim=True)).reshape(-1).to(F32)
    nrm = lambda s, k: torch.randn(k, generator=g, device=DEV, dtype=F64) * s  # noqa: E731
    P = torch.cat([nrm(math.sqrt(2 / FIN), HID * FIN), nrm(0.1, HID), nrm(math.sqrt(2 / HID), HID * HID), nrm(0.1, HID),
                   nrm(math.sqrt(1 / HID), HID), nrm(0.1, 1)]).to(F32)
    m = nrm(0.05, P.shape[0]).to(F32)
    v = (nrm(0.05, P.shape[0]) ** 2 + 1e-4).to(F32)
    goff = (torch.arange(case["groups"] + 1, device=DEV) * case["group_rows"]).to(torch.int32)
    return F, p, P, m, v, goff


def _bf(x):
    return x + (x.float().bfloat16().double() - x).detach()


def _train64(case, seed):
    """The same step in 64 bits, with the network's bfloat16 weights and hidden activations (straight-through)."""
    F, p, P, m, v, goff = (t.double() if t.is_floating_point() else t for t in _train_inputs(case, seed))
    P.requires_grad_(True)
    o = np.cumsum([0, HID * FIN, HID, HID * HID, HID, HID, 1])
    W1, b1, W2, b2, W3, b3 = (P[o[i]:o[i + 1]] for i in range(6))
    loss = torch.zeros((), dtype=F64, device=DEV)
    per = max(1, 65536 // case["group_rows"]) * case["group_rows"]
    gelu = lambda x: 0.5 * x * (1 + torch.tanh(math.sqrt(2 / math.pi) * (x + 0.044715 * x ** 3)))  # noqa: E731
    for a in range(0, F.shape[0], per):
        f, q = F[a:a + per], p[a:a + per].reshape(-1, case["group_rows"])
        h = _bf(gelu(f @ _bf(W1).reshape(HID, FIN).t() + b1))
        h = _bf(gelu(h @ _bf(W2).reshape(HID, HID).t() + b2))
        y = (h @ _bf(W3) + b3).reshape(-1, case["group_rows"])
        part = (q * (q.log() - torch.log_softmax(y, 1))).sum()
        part.backward()
        loss += part.detach()
    g = P.grad
    with torch.no_grad():
        m2, v2 = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        step = 1e-3 * (m2 / (1 - 0.9 ** STEP)) / ((v2 / (1 - 0.999 ** STEP)).sqrt() + 1e-8)
        return {"params": P.detach() - step, "m": m2, "v": v2, "loss": loss.reshape(1)}


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def _context(occluders):
    ctx = api.Context(0)
    ctx.set_occluders(occluders)
    return ctx


def prepare(case, seed):
    kind = case["kind"]
    s = SimpleNamespace(kind=kind)
    if kind == "frame":
        sc = _frame_scene(case, seed)
        s.ctx, s.ds = _context(sc.spheres), api.DeviceScene(sc, DEV)
        s.prm = api.default_params(seed=11, pass1_ppm=case["ppm1"], pass2_ppm=case["ppm2"], learned=case["learned"])
        if case["learned"]:
            w = np.load(os.path.join(os.path.dirname(package.__file__), "proposal_mlp.npy"))
            s.net = torch.as_tensor(w, device=DEV)
            api.set_proposal(s.ctx, s.net)
        coarsen = api.Coarsening(case["draws"], case["n_max"]) if case["draws"] else None
        s.plan = api.Plan(sc, s.prm, coarsen)
        s.ws = api.workspace(s.plan, DEV)
        s.out = torch.empty((sc.m, 3), dtype=F32, device=DEV)
    elif kind == "complete":
        m_s, n1, keys, vals = _samples(case, seed)
        S, n = case["slices"], case["cols"]
        off = np.concatenate([[0], np.cumsum(m_s)]).astype(np.int32)
        layout = SimpleNamespace(n_slices=S, n_clusters=n, pt_offsets=off, rank=np.full(S, case["rank"], np.int32),
                                 cl_offsets=(np.arange(S + 1) * n).astype(np.int32))
        s.ctx, s.prm = api.Context(0), _params(case)
        s.plan = api.Plan(layout, s.prm)
        s.ws = api.workspace(s.plan, DEV)
        api.region_view(s.plan, s.ws, "OMEGA1", torch.int32)[:keys.shape[0]] = keys
        api.region_view(s.plan, s.ws, "VAL1", F32)[:3 * vals.shape[0]] = vals.reshape(-1)
        s.m = int(off[-1])
        s.pt_ids = torch.arange(s.m, dtype=torch.int32, device=DEV)
        s.out = torch.empty((s.m, 3), dtype=F32, device=DEV)
        s.scale = api.region_view(s.plan, s.ws, "SLICE_SCALE", F32)
    elif kind in ("entries", "reference"):
        sc, _, _, _, g = _entry_scene(case, seed)
        s.ctx, s.ds, s.prm = _context(sc.spheres), api.DeviceScene(sc, DEV), api.default_params()
        s.pid, s.lid = _pairs(case, sc, g)
    elif kind == "light_cut":
        sc, _, vpl, _, g = _entry_scene(case, seed)
        perm, _, left, right = _light_tree(vpl[:, :3].double(), vpl.shape[0])
        s.ctx, s.ds = api.Context(0), api.DeviceScene(sc, DEV)
        s.plan = api.LightcutPlan(perm.cpu().numpy(), left, right, case["samples"], case["max_cut"])
        s.ws = s.plan.workspace(DEV)
        s.samples = torch.randperm(sc.m, generator=g, device=DEV)[:case["samples"]].to(torch.int32)
        s.eps = case["eps"]
    else:
        s.F, s.p, s.P, s.m, s.v, s.goff = _train_inputs(case, seed)
        s.ctx, s.step = api.Context(0), STEP
        s.scratch = api.mlp_scratch(s.F.shape[0], DEV)
        s.loss = torch.zeros(1, device=DEV)
    return s


def _pairs(case, sc, g):
    """(point, light) pairs, or the pixels of a reference image."""
    if case["kind"] == "reference":
        return torch.randperm(sc.m, generator=g, device=DEV)[:case["pixels"]].to(torch.int32), None
    r = lambda hi: torch.randint(0, hi, (case["pairs"],), generator=g, device=DEV, dtype=torch.int32)  # noqa: E731
    return r(sc.m), r(sc.n)


def run(s):
    if s.kind == "frame":
        return api.render(s.ctx, s.plan, s.ds, s.prm, s.ws, s.out)
    if s.kind == "complete":
        return {"radiance": api.stage_adm(s.ctx, s.plan, s.prm, s.pt_ids, s.ws, s.m, s.out), "scale": s.scale}
    if s.kind == "entries":
        return api.eval_pairs(s.ctx, s.ds, s.ds.vpl, s.pid, s.lid, s.prm)
    if s.kind == "reference":
        return api.brute_force(s.ctx, s.ds, s.ds.vpl, s.prm, s.pid)
    if s.kind == "light_cut":
        return api.lightcut(s.ctx, s.plan, s.ds, s.samples, s.eps, R_MIN, 5, s.ws)
    api.mlp_train_step(s.ctx, s.P, s.m, s.v, s.step, 1e-3, s.F, s.p, s.goff, s.scratch, s.loss)
    s.step += 1
    return {"params": s.P, "m": s.m, "v": s.v, "loss": s.loss}


def exact(case, seed):
    kind = case["kind"]
    if kind == "complete":
        return _complete64(case, seed)
    if kind == "train":
        return _train64(case, seed)
    if kind in ("entries", "reference"):
        sc, pts, vpl, geo, g = _entry_scene(case, seed)
        pid, lid = _pairs(case, sc, g)
        vis = _visible64(geo[0], sc.spheres)
        if kind == "entries":
            return torch.cat([_shade64(pts[a.long()], vpl[b.long()], vis)
                              for a, b in zip(pid.split(1 << 18), lid.split(1 << 18))])
        out = torch.zeros(pid.shape[0], 3, dtype=F64, device=DEV)
        for a in range(0, pid.shape[0], 256):
            P = pts[pid[a:a + 256].long()]
            for b in range(0, vpl.shape[0], 1024):
                L = vpl[b:b + 1024]
                v = _shade64(P.repeat_interleave(L.shape[0], 0), L.repeat(P.shape[0], 1), vis)
                out[a:a + 256] += v.reshape(P.shape[0], L.shape[0], 3).sum(1)
        return out
    # a frame's integer decisions follow from its 32-bit entries; a cut is whole numbers
    return None


def work(case):
    kind = case["kind"]
    if kind == "frame":
        m, q = case["width"] * case["height"], case["rank"]
        n = case["n_max"] or case["clusters"]
        rows = (m / case["slices"]) if case["slices"] else 0.65 * case["slice_max"]
        S = m / max(1.0, min(rows, m))
        D = rows * n
        deep = math.log2(max(2, case["clusters"]))
        k = min(case["draws"], rows * case["clusters"]) if case["draws"] else 0
        nnz = (0.65 * min(k, D) if k else case["ppm1"] * 1e-6 * D) + case["ppm2"] * 1e-6 * D
        entries = S * (nnz + k * (deep + 1))
        flops = entries * (ENTRY_FLOPS + 0.5 * RAY_FLOPS) + S * 100 * (18.0 * q * nnz + 2.0 * q * q * (4 * rows + 9 * n))
        return {"bytes": m * (POINT_BYTES + 16) + case["vpls"] * (LIGHT_BYTES + 4), "flops": flops}
    if kind == "complete":
        S, n, q = case["slices"], case["cols"], case["rank"]
        lo, hi = case["rows_min"], max(case["rows_max"], case["rows_min"] + 1)
        rows = (hi - lo) / math.log(hi / lo)
        nnz = case["ppm"] * 1e-6 * rows * n
        if case["method"] == "adm":
            it = 18.0 * q * nnz + 2.0 * q * q * (4 * rows + 9 * n)
        else:
            it = nnz * (4.0 * q * q + 12.0 * q + 2.0 * q * q) + (rows + n) * q ** 3 / 3.0 + (rows + 3 * n) * 2.0 * q * q
        return {"bytes": S * (16 * nnz + 16 * rows), "flops": 100.0 * S * it}
    if kind == "entries":
        k = case["pairs"]
        return {"bytes": 20.0 * k + POINT_BYTES * case["points"] + LIGHT_BYTES * case["lights"],
                "flops": k * (ENTRY_FLOPS + 0.5 * RAY_FLOPS)}
    if kind == "reference":
        k = float(case["pixels"]) * case["lights"]
        return {"bytes": case["pixels"] * (POINT_BYTES + 28) + LIGHT_BYTES * case["lights"],
                "flops": k * (ENTRY_FLOPS + 0.5 * RAY_FLOPS)}
    if kind == "light_cut":
        cut = min(case["max_cut"], case["vpls"])
        return {"bytes": case["vpls"] * (LIGHT_BYTES + 16) + case["samples"] * POINT_BYTES + 16.0 * cut,
                "flops": float(case["samples"]) * cut * (2 * ENTRY_FLOPS + 2 * 35)}
    rows = float(case["groups"] * case["group_rows"])
    per = 2.0 * (HID * FIN + HID * HID + HID)
    return {"bytes": rows * 4 * (FIN + 1) + 7 * 4.0 * (HID * FIN + HID * HID + 3 * HID + 1), "flops": 3.0 * per * rows}
