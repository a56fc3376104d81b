// Lighting-matrix entries A(i, j) (Sec. 3): the contribution of a point
// light to a surface point, with a shadow ray against the occluder BVH
// (visibility is the most expensive part of an entry, Sec. 2 and Sec. 6).
//
//   d = y - x, w = d / |d|, c_x = n_x . w, c_y = -n_y . w (0, no ray, if either <= 0)
//   G = c_x c_y / max(|d|^2, r_min^2)
//   f = kd / pi + ks (e + 2) / (2 pi) max(0, w_r . w_o)^e,  w_r = 2 c_x n_x - w
//   A = f * I * G * V
// V = 0 iff the segment from x + eps n_x to y passes within the radius of a
// sphere (closest point of the segment to the centre), found by an any-hit
// traversal of a bounding-volume hierarchy in depth-first order with skip
// indices (no stack).

#include <algorithm>

#include "vplmc_internal.h"
#include "shading.h"

namespace vplmc {
namespace {

// The BVH as read by a traversal: from global memory, or from a copy staged
// in LDS (nodes as pairs of float4, then the spheres).
// KIND: 0 spheres, 1 triangles (Bvh::kind), fixed per kernel instance so that
// the sphere traversal carries no triangle code.
template <int KIND>
struct BvhGlobal {
    static constexpr int kind = KIND;
    const Bvh &b;
    __device__ BvhNode node(int k) const { return b.nodes[k]; }
    __device__ float4 sphere(int k) const { return b.spheres[k]; }
};
template <int KIND>
struct BvhStaged {
    static constexpr int kind = KIND;
    const float4 *lds;   // LDS: 2 n_nodes float4 of nodes, then the spheres or triangles
    int n_nodes;
    __device__ BvhNode node(int k) const {
        const float4 a = lds[2 * k], c = lds[2 * k + 1];
        BvhNode nd;
        nd.lo[0] = a.x;
        nd.lo[1] = a.y;
        nd.lo[2] = a.z;
        nd.leaf = __float_as_int(a.w);
        nd.hi[0] = c.x;
        nd.hi[1] = c.y;
        nd.hi[2] = c.z;
        nd.skip = __float_as_int(c.w);
        return nd;
    }
    __device__ float4 sphere(int k) const { return lds[2 * n_nodes + k]; }
};

// does a triangle reference of a leaf meet the open segment o + t D,
// t in (0, 1): barycentric u, v >= 0, u + v <= 1 of the crossing with the
// triangle's plane (Moller-Trumbore), none for a segment parallel to it
template <typename B>
__device__ __forceinline__ bool leaf_occludes_tri(const B &bvh, int first, int cnt, P3 o, P3 D) {
    bool any = false;
    for (int k = 0; k < cnt; ++k) {
        const float4 a4 = bvh.sphere(3 * (first + k)), b4 = bvh.sphere(3 * (first + k) + 1);
        const float4 c4 = bvh.sphere(3 * (first + k) + 2);
        const P3 e1 = {b4.x, b4.y, b4.z}, e2 = {c4.x, c4.y, c4.z};
        const P3 p = {D.y * e2.z - D.z * e2.y, D.z * e2.x - D.x * e2.z, D.x * e2.y - D.y * e2.x};
        const float det = dot(e1, p);
        const float inv = 1.0f / det;
        const P3 s = {o.x - a4.x, o.y - a4.y, o.z - a4.z};
        const float u = dot(s, p) * inv;
        const P3 q = {s.y * e1.z - s.z * e1.y, s.z * e1.x - s.x * e1.z, s.x * e1.y - s.y * e1.x};
        const float v = dot(D, q) * inv;
        const float t = dot(e2, q) * inv;
        any = any || (det != 0.0f && u >= 0.0f && v >= 0.0f && u + v <= 1.0f && t > 0.0f && t < 1.0f);
    }
    return any;
}

// does a sphere of a leaf (first << 4 | count) come closer to the segment
// o + t D, t in [0, 1], than its radius (or, for triangle occluders, does a
// triangle of the leaf meet it)
template <typename B>
__device__ __forceinline__ bool leaf_occludes(const B &bvh, int leaf, P3 o, P3 D, float inv_dd) {
    const int first = leaf >> 4, cnt = leaf & 15;
    if constexpr (B::kind == 1) return leaf_occludes_tri(bvh, first, cnt, o, D);
    bool any = false;
    for (int k = 0; k < cnt; ++k) {
        const float4 sp4 = bvh.sphere(first + k);
        const P3 oc = {sp4.x - o.x, sp4.y - o.y, sp4.z - o.z};
        const float t = fminf(fmaxf(dot(oc, D) * inv_dd, 0.0f), 1.0f);
        const P3 p = {oc.x - t * D.x, oc.y - t * D.y, oc.z - t * D.z};
        any = any || dot(p, p) < sp4.w * sp4.w;
    }
    return any;
}

// any hit on the open segment o + t D, t in (0, 1)
template <typename B>
__device__ __forceinline__ bool occluded_in(const B &bvh, int n_nodes, P3 o, P3 D) {
    if (n_nodes == 0) return false;
    const float dd = dot(D, D);
    const float inv_dd = 1.0f / dd;
    const float ix = 1.0f / (fabsf(D.x) > 1e-20f ? D.x : copysignf(1e-20f, D.x));
    const float iy = 1.0f / (fabsf(D.y) > 1e-20f ? D.y : copysignf(1e-20f, D.y));
    const float iz = 1.0f / (fabsf(D.z) > 1e-20f ? D.z : copysignf(1e-20f, D.z));
    int node = 0;
    while (node < n_nodes) {
        const BvhNode nd = bvh.node(node);
        const float tx0 = (nd.lo[0] - o.x) * ix, tx1 = (nd.hi[0] - o.x) * ix;
        const float ty0 = (nd.lo[1] - o.y) * iy, ty1 = (nd.hi[1] - o.y) * iy;
        const float tz0 = (nd.lo[2] - o.z) * iz, tz1 = (nd.hi[2] - o.z) * iz;
        const float tmin = fmaxf(fmaxf(fminf(tx0, tx1), fminf(ty0, ty1)), fmaxf(fminf(tz0, tz1), 0.0f));
        const float tmax = fminf(fminf(fmaxf(tx0, tx1), fmaxf(ty0, ty1)), fminf(fmaxf(tz0, tz1), 1.0f));
        const bool hit = tmin <= tmax;
        if (hit && nd.leaf != 0 && leaf_occludes(bvh, nd.leaf, o, D, inv_dd)) return true;
        // an inner node that is hit descends to its left child; anything else
        // continues after its subtree
        node = hit && nd.leaf == 0 ? node + 1 : nd.skip;
    }
    return false;
}


// entry of one (point, light) pair (zero when the pair faces away or is
// occluded); bvh is a BVH view (BvhGlobal or BvhStaged) of n_nodes nodes.
// Returns whether a shadow ray was cast (both cosines positive).
template <typename B>
__device__ __forceinline__ bool shade_in(const B &bvh, int n_nodes, const PointData &q, const Light &L,
                                         float r_min2, float eps, float &o0, float &o1, float &o2) {
    o0 = o1 = o2 = 0.0f;
    const P3 d = sub(L.y, q.x);
    const float r2 = dot(d, d);
    const float inv_r = 1.0f / sqrtf(r2);
    const P3 w = {d.x * inv_r, d.y * inv_r, d.z * inv_r};
    const float cx = dot(q.n, w);
    const float cy = -dot(L.n, w);
    if (!(cx > 0.0f && cy > 0.0f)) return false;
    const float G = cx * cy / fmaxf(r2, r_min2);
    float spec = 0.0f;
    if (q.ks > 0.0f) {
        const P3 wr = {2.0f * cx * q.n.x - w.x, 2.0f * cx * q.n.y - w.y, 2.0f * cx * q.n.z - w.z};
        const float cr = fmaxf(0.0f, dot(wr, q.wo));
        spec = q.ks * (q.e + 2.0f) * (0.5f * INV_PI) * powf(cr, q.e);
    }
    const P3 o = {fmaf(eps, q.n.x, q.x.x), fmaf(eps, q.n.y, q.x.y), fmaf(eps, q.n.z, q.x.z)};
    if (occluded_in(bvh, n_nodes, o, sub(L.y, o))) return true;
    o0 = fmaf(q.kd0, INV_PI, spec) * L.i0 * G;
    o1 = fmaf(q.kd1, INV_PI, spec) * L.i1 * G;
    o2 = fmaf(q.kd2, INV_PI, spec) * L.i2 * G;
    return true;
}

template <int KIND>
__device__ __forceinline__ bool shade(const Bvh &bvh, const PointData &q, const Light &L, float r_min2,
                                      float eps, float &o0, float &o1, float &o2) {
    return shade_in(BvhGlobal<KIND>{bvh}, bvh.n_nodes, q, L, r_min2, eps, o0, o1, o2);
}

// LDS written by some lanes of a wavefront and then read by others
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// minimum over the wavefront, uniform
__device__ __forceinline__ float wave_min(float v) {
    v = fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true)));
    v = fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true)));
    v = fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, true)));
    v = fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xF, 0xF, true)));
    const int b = __float_as_int(v);
    return fminf(fminf(__int_as_float(__builtin_amdgcn_readlane(b, 0)), __int_as_float(__builtin_amdgcn_readlane(b, 16))),
                 fminf(__int_as_float(__builtin_amdgcn_readlane(b, 32)), __int_as_float(__builtin_amdgcn_readlane(b, 48))));
}

// Shadow segments of a whole wavefront against the spheres near their common
// shaft.  The segments of lanes with `want` run from o, inside the box A of
// their origins, to y, inside the box B of their ends; at parameter t every
// one of them is inside the box between A and B at t, so a sphere can only be
// met if its box overlaps that moving box for some t in [0, 1], six linear
// conditions on t.  The lanes test a box each: the groups of BVH_GROUP
// consecutive (hence close) spheres, 64 at a time, then the spheres of the
// groups that pass, two groups at a time; the spheres that pass are listed in
// LDS, and every lane tests its own segment against the list exactly as a BVH
// leaf does.  All boxes are padded beyond FP32 rounding, so the list holds
// every sphere that any of the segments meets and the answer is that of the
// traversal.  It pays where the segments of a wavefront are alike: rows of one
// slice against one light or the lights below one tree node.  Returns 1
// (occluded), 0 (not), or -1 for every lane if the list overflows or a segment
// starts beyond any box.  All 64 lanes call.
constexpr int SHAFT_CAP = 128;
// The tests of the groups are linear in their number; a traversal is not.  8,192
// points against 4,096 lights and fine spheres, lists / traversal of the same
// wavefronts: 1,024 groups 8.1 / 7.9 ms, 2,048 groups 10.2 / 10.1 ms.  Spheres that
// cover the same part of the scene whatever their number: 128 groups 3.56 / 3.97 ms,
// 256 4.74 / 4.70, 512 4.82 / 4.75, 1,024 5.09 / 5.00; 512 x 512 coarsened frames
// 24.8 / 24.9, 26.6 / 26.3, 27.9 / 27.5, 29.4 / 28.9 ms.
constexpr int SHAFT_MAX_GROUPS = 512;

// an origin that the arithmetic on boxes takes (an infinite one would leave every lane of its wavefront an empty shaft)
__device__ __forceinline__ bool boxed(P3 o) { return fabsf(o.x) < 1e18f && fabsf(o.y) < 1e18f && fabsf(o.z) < 1e18f; }

// the spheres near the shaft between the boxes A and B (wave-uniform) listed in
// `list`; their number, or one above SHAFT_CAP if that many do not fit
__device__ __forceinline__ int shaft_list(const Bvh &b, float4 *list, float (&alo)[3], float (&ahi)[3],
                                          const float (&blo)[3], const float (&bhi)[3]) {
    const int lane = threadIdx.x & 63;
    float ilo[3], ihi[3], slo[3], shi[3];   // lines of the lower and upper box sides (from alo, ahi): 1 / slope, sign
    float big = 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        big = fmaxf(fmaxf(big, fmaxf(fabsf(alo[k]), fabsf(ahi[k]))), fmaxf(fabsf(blo[k]), fabsf(bhi[k])));
    const float pad = 1e-5f * big;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float dl = blo[k] - alo[k], dh = bhi[k] - ahi[k];
        alo[k] -= pad;
        ahi[k] += pad;
        ilo[k] = 1.0f / (fabsf(dl) > 1e-20f ? dl : copysignf(1e-20f, dl));
        ihi[k] = 1.0f / (fabsf(dh) > 1e-20f ? dh : copysignf(1e-20f, dh));
        slo[k] = ilo[k] > 0.f ? -INFINITY : INFINITY;
        shi[k] = ihi[k] > 0.f ? -INFINITY : INFINITY;
    }
    // does the box [lo, hi] overlap the moving box at some t in [0, 1]:
    // alo + t dl <= hi and ahi + t dh >= lo on every axis
    auto meets = [&](const float (&lo)[3], const float (&hi)[3]) {
        float t0 = -1e-5f, t1 = 1.0f + 1e-5f;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float u = (hi[k] - alo[k]) * ilo[k];        // upper bound of t on a rising side, lower on a falling one
            t1 = fminf(t1, fmaxf(u, slo[k]));
            t0 = fmaxf(t0, fminf(u, slo[k]));
            const float v = (lo[k] - ahi[k]) * ihi[k];
            t0 = fmaxf(t0, fminf(v, -shi[k]));
            t1 = fminf(t1, fmaxf(v, -shi[k]));
        }
        return t0 <= t1 + 1e-5f;
    };
    int count = 0;
    // (ending within 64 groups as well saved 1-2% where lists overflow and cost 2-4% where they do not)
    for (int g0 = 0; g0 < b.n_groups && count <= SHAFT_CAP; g0 += 64) {
        bool in = false;
        if (g0 + lane < b.n_groups) {
            const float4 l4 = b.groups[2 * (g0 + lane)], h4 = b.groups[2 * (g0 + lane) + 1];
            const float lo[3] = {l4.x, l4.y, l4.z}, hi[3] = {h4.x, h4.y, h4.z};
            in = meets(lo, hi);
        }
        unsigned long long mask = __ballot(in);
        while (mask) {
            const int ga = g0 + __ffsll(mask) - 1;
            mask &= mask - 1;
            const int gb = mask ? g0 + __ffsll(mask) - 1 : -1;
            mask = mask ? mask & (mask - 1) : 0;
            const int e = (lane < 32 ? ga : gb) * BVH_GROUP + lane % 32;
            bool hit = false;
            float4 sp = make_float4(0.f, 0.f, 0.f, 0.f);
            if (e >= 0 && e < b.n_spheres) {
                sp = b.spheres[e];
                const float rr = fmaf(1e-6f, fabsf(sp.x) + fabsf(sp.y) + fabsf(sp.z), 1.00001f * sp.w);
                const float lo[3] = {sp.x - rr, sp.y - rr, sp.z - rr}, hi[3] = {sp.x + rr, sp.y + rr, sp.z + rr};
                hit = meets(lo, hi);
            }
            const unsigned long long hits = __ballot(hit);
            const int at = count + __popcll(hits & ((1ull << lane) - 1));
            if (hit && at < SHAFT_CAP) list[at] = sp;
            count += __popcll(hits);
        }
    }
    return count;
}

// is the lane's segment from o to y met by one of the first `count` listed spheres
__device__ __forceinline__ bool list_occluded(const float4 *list, int count, bool want, P3 o, P3 y) {
    wave_lds_sync();
    const P3 D = sub(y, o);
    const float inv_dd = 1.0f / dot(D, D);
    bool occ = false;
    for (int k0 = 0; k0 < count; k0 += 8) {
        for (int k = k0; k < min(count, k0 + 8); ++k) {
            const float4 sp4 = list[k];
            const P3 oc = {sp4.x - o.x, sp4.y - o.y, sp4.z - o.z};
            const float t = fminf(fmaxf(dot(oc, D) * inv_dd, 0.0f), 1.0f);
            const P3 p = {oc.x - t * D.x, oc.y - t * D.y, oc.z - t * D.z};
            occ = occ || dot(p, p) < sp4.w * sp4.w;
        }
        if (__ballot(want && !occ) == 0) break;
    }
    wave_lds_sync();             // the next list overwrites this one
    return want && occ;
}

// Whether a wavefront lists at all: after a list that overflowed it traverses the
// BVH for the next 1, 2, 4, ... SHAFT_BACKOFF segments of each lane, so that
// dense occluders cost a few failed lists per wavefront instead of one per tree level.
constexpr int SHAFT_BACKOFF = 64;
struct ShaftGate {
    int wait = 0, penalty = 0;
    __device__ bool open() {
        if (wait == 0) return true;
        --wait;
        return false;
    }
    __device__ void listed(bool fits) {
        penalty = fits ? 0 : min(max(1, 2 * penalty), SHAFT_BACKOFF);
        wait = penalty;
    }
};

__device__ int occluded_shaft(const Bvh &b, float4 *list, ShaftGate &gate, bool want, P3 o, P3 y) {
    if (b.n_groups == 0 || __ballot(want) == 0) return 0;
    if (!gate.open() || __ballot(want && !boxed(o)) != 0) return -1;
    const float of[3] = {o.x, o.y, o.z}, yf[3] = {y.x, y.y, y.z};
    float alo[3], ahi[3], blo[3], bhi[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        alo[k] = wave_min(want ? of[k] : INFINITY);
        ahi[k] = -wave_min(want ? -of[k] : INFINITY);
        blo[k] = wave_min(want ? yf[k] : INFINITY);
        bhi[k] = -wave_min(want ? -yf[k] : INFINITY);
    }
    const int count = shaft_list(b, list, alo, ahi, blo, bhi);
    gate.listed(count <= SHAFT_CAP);
    if (count > SHAFT_CAP) return -1;
    return list_occluded(list, count, want, o, y) ? 1 : 0;
}

// shade_in for a whole wavefront (all 64 lanes call; lanes without `on` get zeros)
template <int KIND, typename S>
__device__ __forceinline__ bool shade_wave(const Bvh &bvh, const S *staged, float4 *list, ShaftGate &gate, bool on,
                                           const PointData &q, const Light &L, float r_min2, float eps, float &o0, float &o1, float &o2) {
    if constexpr (KIND == 0) {
        o0 = o1 = o2 = 0.f;
        bool ray = false;
        if (on) ray = entry_unoccluded(q, L, r_min2, o0, o1, o2);
        const P3 o = {fmaf(eps, q.n.x, q.x.x), fmaf(eps, q.n.y, q.x.y), fmaf(eps, q.n.z, q.x.z)};
        int occ = bvh.n_groups <= SHAFT_MAX_GROUPS ? occluded_shaft(bvh, list, gate, ray, o, L.y) : -1;
        if (occ < 0) occ = ray && occluded_in(BvhGlobal<KIND>{bvh}, bvh.n_nodes, o, sub(L.y, o)) ? 1 : 0;
        if (occ) o0 = o1 = o2 = 0.f;
        return ray;
    } else {
        bool ray = false;
        o0 = o1 = o2 = 0.f;
        if (on) {
            if (staged) ray = shade_in(*staged, bvh.n_nodes, q, L, r_min2, eps, o0, o1, o2);
            else ray = shade<KIND>(bvh, q, L, r_min2, eps, o0, o1, o2);
        }
        return ray;
    }
}

// adds a per-thread count into a device total: one atomic per wavefront
__device__ __forceinline__ void add_count(unsigned long long *total, uint32_t v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0 && v) atomicAdd(total, (unsigned long long)v);
}

__device__ __forceinline__ int slice_of_off(const SliceDesc *__restrict__ desc, int S, int64_t g, int which) {
    int lo = 0, hi = S;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        const int64_t o = which ? desc[mid].off2 : desc[mid].off1;
        if (o <= g) lo = mid; else hi = mid;
    }
    return lo;
}

// entry of sample g of one pass (nothing for slots past the slice's first-pass
// count or its accepted second-pass count)
template <bool STAGED, int KIND>
__device__ __forceinline__ uint32_t eval_one(const Bvh &bvh, const BvhStaged<KIND> &staged, const vplmc_points &pts,
                                         const float *__restrict__ lights, int32_t n_lights,
                                         const SliceDesc *__restrict__ desc, int S, const int32_t *__restrict__ pt_ids,
                                         const int32_t *__restrict__ cl_ids, const uint32_t *__restrict__ keys,
                                         int64_t g, int which, const int32_t *__restrict__ stats, float r_min2,
                                         float eps, float *__restrict__ vals) {
    const int s = slice_of_off(desc, S, g, which);
    const SliceDesc d = desc[s];
    if (which ? g - d.off2 >= stats[4 * s + 3] : g - d.off1 >= d.N1) return 0;
    const uint32_t key = keys[g];
    const int i = (int)(key >> 16), j = (int)(key & 0xFFFFu);
    const int pid = pt_ids[d.pt_off + i];
    const int c = clamp_index(cl_ids[d.cl_off + j], n_lights);
    const size_t N = (size_t)n_lights;
    const Light L = {{lights[c], lights[N + c], lights[2 * N + c]},
                     {lights[3 * N + c], lights[4 * N + c], lights[5 * N + c]},
                     lights[6 * N + c], lights[7 * N + c], lights[8 * N + c]};
    const PointData q = load_point(pts, pid);
    float o0, o1, o2;
    bool ray;
    if (STAGED)
        ray = shade_in(staged, bvh.n_nodes, q, L, r_min2, eps, o0, o1, o2);
    else
        ray = shade<KIND>(bvh, q, L, r_min2, eps, o0, o1, o2);
    vals[3 * g] = o0;
    vals[3 * g + 1] = o1;
    vals[3 * g + 2] = o2;
    return ray ? 1u : 0u;
}

// BVH bytes (nodes and spheres) an entry kernel stages in LDS; larger ones are
// read from global memory
constexpr int EVAL_LDS_BYTES = 48 * 1024;
// workgroups per compute unit of an entry launch
constexpr int EVAL_GRID_PER_CU = 16;

// entries of one pass's samples (draw order), lights = cluster table planes;
// a fixed grid walks the samples, each workgroup first copying the BVH to LDS
// when STAGED
template <bool STAGED, int KIND>
__global__ __launch_bounds__(256) void k_eval_omega(Bvh bvh, vplmc_points pts, const float *__restrict__ lights,
                                                    int32_t n_lights, const SliceDesc *__restrict__ desc, int S,
                                                    const int32_t *__restrict__ pt_ids,
                                                    const int32_t *__restrict__ cl_ids,
                                                    const uint32_t *__restrict__ keys, int64_t n_keys,
                                                    int which, const int32_t *__restrict__ stats, float r_min2,
                                                    float eps, float *__restrict__ vals,
                                                    unsigned long long *__restrict__ rays) {
    extern __shared__ float4 stage[];
    if (STAGED) {
        const int nn = 2 * bvh.n_nodes, ns = bvh.n_spheres;
        const float4 *nodes4 = reinterpret_cast<const float4 *>(bvh.nodes);
        for (int k = threadIdx.x; k < nn + ns; k += blockDim.x) stage[k] = k < nn ? nodes4[k] : bvh.spheres[k - nn];
        __syncthreads();
    }
    const BvhStaged<KIND> staged{stage, bvh.n_nodes};
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    uint32_t traced = 0;
    for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < n_keys; g += stride) {
        traced += eval_one<STAGED, KIND>(bvh, staged, pts, lights, n_lights, desc, S, pt_ids, cl_ids, keys, g, which, stats,
                                   r_min2, eps, vals);
    }
    if (rays) add_count(rays, traced);
}

// Merge errors of the per-slice light coarsening (Sec. 4).  One thread per
// row draw (slice s, draw r; r < kpre[n_g]): draw k < m' of leaf x, its row
// the k-th image of leaf x's keyed permutation of [0, m') (4-round
// Feistel, round function Philox(key = (seed, s), ctr = (R, round, TAG_ZETA,
// x)) & mask, cycle-walked).  Walking from x to the root, the thread carries
// S(i, rep of the current node) at unit intensity; at each split node f
// (kept child a, dropped b) one new entry gives the other child's, and
// I_b |S(i, rep_b) - S(i, rep_a)| (max over channels) goes into eps(f) by an
// integer max (non-negative floats order as their bits).  A node's light is
// its kept child's, so the carried value becomes S(i, rep_a).  Every node's
// eps is thus the max over the union of its leaves' draws, each pixel
// evaluated once per level (the reuse Sec. 4 describes).
__device__ __forceinline__ uint64_t feistel_zeta(uint64_t v, uint64_t seed, uint64_t s, uint64_t x, int h) {
    const uint64_t mask = (1ull << h) - 1ull;
    uint64_t L = v >> h, R = v & mask;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint64_t F = philox(seed, s, R, (uint64_t)r, TAG_ZETA, x).a & mask;
        const uint64_t nL = R;
        R = L ^ F;
        L = nL;
    }
    return (L << h) | R;
}


// the row of draw k of leaf x in slice s of m rows
__device__ __forceinline__ int draw_row(int64_t k, int32_t rows, uint64_t seed, int s, int x) {
    const uint64_t m = (uint64_t)rows;
    int b = m > 1 ? 64 - __clzll((long long)(m - 1)) : 0;
    b = b < 2 ? 2 : b;
    const int h = (b + 1) / 2;
    uint64_t e = feistel_zeta((uint64_t)k, seed, (uint64_t)s, (uint64_t)x, h);
    while (e >= m) e = feistel_zeta(e, seed, (uint64_t)s, (uint64_t)x, h);
    return (int)e;
}

__device__ __forceinline__ void raise_error(float *slot_f, float err) {
    unsigned int *slot = reinterpret_cast<unsigned int *>(slot_f);
    const unsigned int bits = __float_as_uint(err);
    if (__hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < bits) atomicMax(slot, bits);
}

// whether the lights of the top of the tree are taken from a table: only where
// at least half of the nominal draws exist (with fewer draws than leaves most
// quotas round down to none)
__device__ __forceinline__ bool top_table(const CoarsenTree &tr, const CoarsenSlices &cs, int64_t K) {
    return tr.n_front > 1 && 2 * cs.kpre[tr.n_leaves] >= K;
}

// The walk of few draws: every thread its own path to the root, draws in leaf-id
// order, the occluders staged in LDS where they fit.
// Six wavefronts per SIMD (80 VGPRs): the walk's latency needs the occupancy;
// at 83 VGPRs (five) the kernel ran 14% slower on the 1080p frame.
template <bool STAGED, int KIND>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6, 8))) void k_coarsen_walk(
    Bvh bvh, vplmc_points pts, const float *__restrict__ lights, const SliceDesc *__restrict__ desc, int64_t total, int64_t K,
    const int32_t *__restrict__ pt_ids, CoarsenTree tr, CoarsenSlices cs, uint64_t seed, float r_min2, float eps,
    unsigned long long *__restrict__ counts) {
    extern __shared__ float4 stage[];
    if (STAGED) {
        const int nn = 2 * bvh.n_nodes, ns = bvh.n_spheres;
        const float4 *nodes4 = reinterpret_cast<const float4 *>(bvh.nodes);
        for (int k = threadIdx.x; k < nn + ns; k += blockDim.x) stage[k] = k < nn ? nodes4[k] : bvh.spheres[k - nn];
        __syncthreads();
    }
    const BvhStaged<KIND> staged{stage, bvh.n_nodes};
    const int ng = tr.n_leaves;
    const size_t N = (size_t)(2 * ng - 1);
    const int64_t kt = cs.kpre[ng];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    uint32_t n_eval = 0, n_ray = 0;
    for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < total; g += stride) {
        const int s = (int)(g / K);
        const int64_t r = g - (int64_t)s * K;
        if (r >= kt) continue;
        const SliceDesc d = desc[s];
        int lo = 0, hi = ng;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (cs.kpre[mid] <= r) lo = mid; else hi = mid;
        }
        const int x = lo;
        const int64_t k = r - cs.kpre[x];
        if (k >= d.m) continue;
        const int i = draw_row(k, d.m, seed, s, x);
        cs.zeta[g] = (uint16_t)i;
        const PointData q = load_point(pts, pt_ids[d.pt_off + i]);
        auto entry = [&](int c, float &o0, float &o1, float &o2) {
            const Light L = node_light(lights, N, c, true);
            const bool ray = STAGED ? shade_in(staged, bvh.n_nodes, q, L, r_min2, eps, o0, o1, o2)
                                    : shade<KIND>(bvh, q, L, r_min2, eps, o0, o1, o2);
            n_eval += 1;
            n_ray += ray ? 1u : 0u;
        };
        float c0, c1, c2;
        entry(x, c0, c1, c2);
        float *node_eps = cs.eps + (size_t)s * (ng - 1);
        int c = x;
        for (int f = tr.parent[x]; f >= 0; c = f, f = tr.parent[f]) {
            const int kk = f - ng;
            const int a = cs.kept[kk], bb = cs.dropped[kk];
            const bool kept_path = c == a;
            float o0, o1, o2;
            entry(kept_path ? bb : a, o0, o1, o2);
            const float a0 = kept_path ? c0 : o0, a1 = kept_path ? c1 : o1, a2 = kept_path ? c2 : o2;
            const float b0 = kept_path ? o0 : c0, b1 = kept_path ? o1 : c1, b2 = kept_path ? o2 : c2;
            const float err = fmaxf(fmaxf(lights[6 * N + bb] * fabsf(b0 - a0), lights[7 * N + bb] * fabsf(b1 - a1)),
                                    lights[8 * N + bb] * fabsf(b2 - a2));
            if (err > 0.0f) raise_error(node_eps + kk, err);
            c0 = a0;
            c1 = a1;
            c2 = a2;
        }
    }
    if (counts) {
        add_count(counts, n_eval);
        add_count(counts + 1, n_ray);
    }
}

// The top of the tree, where the draws below a node outnumber the slice's rows
// and the walk would evaluate the same (row, light) many times: every row of a
// run of slices against the lights of the front nodes, once each.  Lanes are
// consecutive rows of a slice against one light, so their shadow rays are alike.
constexpr int TOP_LIGHTS = 8;    // front nodes per thread
template <bool STAGED, int KIND>
__global__ __launch_bounds__(256) void k_coarsen_top(Bvh bvh, vplmc_points pts, const float *__restrict__ lights,
                                                     const SliceDesc *__restrict__ desc, int32_t s_first, int32_t s_end,
                                                     int64_t row_first, int64_t rows, int64_t K,
                                                     const int32_t *__restrict__ pt_ids, CoarsenTree tr, CoarsenSlices cs,
                                                     float r_min2, float eps) {
    extern __shared__ float4 stage[];
    if (STAGED) {
        const int nn = 2 * bvh.n_nodes, ns = bvh.n_spheres;
        const float4 *nodes4 = reinterpret_cast<const float4 *>(bvh.nodes);
        for (int k = threadIdx.x; k < nn + ns; k += blockDim.x) stage[k] = k < nn ? nodes4[k] : bvh.spheres[k - nn];
        __syncthreads();
    }
    const BvhStaged<KIND> staged{stage, bvh.n_nodes};
    __shared__ float4 lists[KIND == 0 ? 256 / 64 * SHAFT_CAP : 1];
    float4 *list = lists + (KIND == 0 ? threadIdx.x / 64 * SHAFT_CAP : 0);
    ShaftGate gate;
    if (!top_table(tr, cs, K)) return;
    const int64_t R0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const bool act = R0 < rows;
    const int64_t R = act ? R0 : rows - 1;
    int lo = s_first, hi = s_end;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (desc[mid].off_row - mid - row_first <= R) lo = mid; else hi = mid;
    }
    const SliceDesc d = desc[lo];
    const int64_t base = d.off_row - lo - row_first;
    const int i = (int)(R - base);
    const PointData q = load_point(pts, pt_ids[d.pt_off + i]);
    float4 *out = cs.top_val + base * tr.n_front + i;
    const size_t N = (size_t)(2 * tr.n_leaves - 1);
    const int k1 = min(tr.n_front, (int)(blockIdx.y + 1) * TOP_LIGHTS);
    for (int k = blockIdx.y * TOP_LIGHTS; k < k1; ++k) {
        float o0, o1, o2;
        const bool ray = shade_wave<KIND>(bvh, STAGED ? &staged : nullptr, list, gate, act, q,
                                          node_light(lights, N, tr.front[k], true), r_min2, eps, o0, o1, o2);
        if (act) out[(int64_t)k * d.m] = make_float4(o0, o1, o2, ray ? 1.f : 0.f);
    }
}

// The walk of many draws: in depth-first order of their leaves (dpre, the prefix
// of the draw counts in that order), so that the lanes of a wavefront lie below
// one small subtree, and all lanes on one tree level at a time (deeper leaves start
// earlier), so that they meet the same node's light as soon as they are below it:
// their shadow rays share a candidate list (occluded_shaft), and one lane adds
// the largest of their errors.  Lights of the top of the tree come from
// k_coarsen_top's table.  Bound by VALU work (0.81 busy):
// shading a third, shadow tests a third, the draws' permutation a ninth.
// Measured on one MI355X, 1080p frame (3,069 slices, 32,768 draws, 16,384
// leaves, 2,048 spheres): 154 ms with draws in leaf-id order, 135 depth-first,
// 114 + 7.4 with the top of the tree evaluated once per row, 49.7 + 2.9 with
// the shared candidate lists.  Measured and not kept: a wavefront walking the
// BVH together with scalar loads (162), leaf tests postponed until few lanes
// still walk (145-174), four wavefronts per SIMD (52.3; five and six alike).
template <bool STAGED, int KIND>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5, 8))) void k_coarsen_eps(Bvh bvh, vplmc_points pts, const float *__restrict__ lights,
                                                     const SliceDesc *__restrict__ desc, int32_t s_first, int64_t row_first,
                                                     int64_t total, int64_t K, const int32_t *__restrict__ pt_ids, CoarsenTree tr,
                                                     CoarsenSlices cs, uint64_t seed, float r_min2, float eps,
                                                     unsigned long long *__restrict__ counts) {
    extern __shared__ float4 stage[];
    if (STAGED) {
        const int nn = 2 * bvh.n_nodes, ns = bvh.n_spheres;
        const float4 *nodes4 = reinterpret_cast<const float4 *>(bvh.nodes);
        for (int k = threadIdx.x; k < nn + ns; k += blockDim.x) stage[k] = k < nn ? nodes4[k] : bvh.spheres[k - nn];
        __syncthreads();
    }
    const BvhStaged<KIND> staged{stage, bvh.n_nodes};
    const int ng = tr.n_leaves;
    const size_t N = (size_t)(2 * ng - 1);
    const int64_t kt = cs.kpre[ng];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    uint32_t n_eval = 0, n_ray = 0;
    const int lane = threadIdx.x & 63;
    const bool table = top_table(tr, cs, K);
    __shared__ float4 lists[KIND == 0 ? 256 / 64 * SHAFT_CAP : 1];
    float4 *list = lists + (KIND == 0 ? threadIdx.x / 64 * SHAFT_CAP : 0);
    ShaftGate gate;
    for (int64_t base = blockIdx.x * (int64_t)blockDim.x + (threadIdx.x - lane); base < total; base += stride) {
        const int64_t g = base + lane < total ? base + lane : total - 1;
        const int sl = (int)(g / K), s = s_first + sl;
        const int64_t r = g - (int64_t)sl * K;
        const SliceDesc d = desc[s];
        // draw r of the slice in depth-first leaf order
        int lo = 0, hi = ng;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (cs.dpre[mid] <= r) lo = mid; else hi = mid;
        }
        const int x = tr.dfs[lo];
        const int64_t k = r - cs.dpre[lo];
        const bool act = base + lane < total && r < kt && k < d.m;
        if (__ballot(act) == 0) continue;
        int i = 0;
        if (act) {
            i = draw_row(k, d.m, seed, s, x);
            cs.zeta[(int64_t)s * K + cs.kpre[x] + k] = (uint16_t)i;
        }
        const PointData q = load_point(pts, pt_ids[d.pt_off + i]);
        // levels from the deepest leaf of the wavefront up, all lanes on one
        // level: lanes below one node evaluate the same light
        const int dep = act ? tr.depth[lo] : -1;
        int level = dep;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) level = max(level, __shfl_xor(level, o, 64));
        const float4 *top = cs.top_val + (d.off_row - s - row_first) * tr.n_front + i;   // the row's entry of front node k: top[k m]
        float *node_eps = cs.eps + (size_t)s * (ng - 1);
        float c0 = 0.f, c1 = 0.f, c2 = 0.f;
        int c = x;
        for (level = __builtin_amdgcn_readfirstlane(level); level >= 0; --level) {
            const bool on = level <= dep;
            // the lane's leaf itself, then the other child of each ancestor
            const bool first = level == dep, up = on && !first;
            const int f = up ? tr.parent[c] : ng;
            const int kk = f - ng;
            const int a = up ? cs.kept[kk] : x, bb = up ? cs.dropped[kk] : x;
            const int other = c == a ? bb : a;
            float o0, o1, o2;
            const int ti = table && on ? tr.tidx[other] : -1;
            bool ray = shade_wave<KIND>(bvh, STAGED ? &staged : nullptr, list, gate, on && ti < 0, q,
                                        node_light(lights, N, other, true), r_min2, eps, o0, o1, o2);
            if (ti >= 0) {                       // in the top of the tree: evaluated by k_coarsen_top
                const float4 v = top[(int64_t)cs.top_map[ti] * d.m];
                o0 = v.x;
                o1 = v.y;
                o2 = v.z;
                ray = v.w != 0.f;
            }
            n_eval += on ? 1u : 0u;
            n_ray += on && ray ? 1u : 0u;
            const bool kept_path = c == a;
            const float a0 = kept_path ? c0 : o0, a1 = kept_path ? c1 : o1, a2 = kept_path ? c2 : o2;
            const float b0 = kept_path ? o0 : c0, b1 = kept_path ? o1 : c1, b2 = kept_path ? o2 : c2;
            const float e = fmaxf(fmaxf(lights[6 * N + bb] * fabsf(b0 - a0), lights[7 * N + bb] * fabsf(b1 - a1)),
                                  lights[8 * N + bb] * fabsf(b2 - a2));
            const float err = up ? e : 0.f;
            const unsigned long long some = __ballot(err > 0.0f);
            if (some) {
                const int lead = __ffsll(some) - 1;
                const int k1 = __builtin_amdgcn_readlane(kk, lead), s1 = __builtin_amdgcn_readlane(s, lead);
                // lanes below one node of one slice: their largest only
                const bool one = __ballot(err > 0.0f && (kk != k1 || s != s1)) == 0;
                const float top_err = one ? -wave_min(err > 0.0f ? -err : 0.f) : err;
                if (one ? lane == lead : err > 0.0f) raise_error(node_eps + kk, top_err);
            }
            if (on) {
                c0 = first ? o0 : a0;
                c1 = first ? o1 : a1;
                c2 = first ? o2 : a2;
                c = first ? c : f;
            }
        }
    }
    if (counts) {
        add_count(counts, n_eval);
        add_count(counts + 1, n_ray);
    }
}

// every entry of one slice, row-major: out[(i n + j) 3 + c]
template <int KIND>
__global__ __launch_bounds__(256) void k_full_matrix(Bvh bvh, vplmc_points pts, const float *__restrict__ lights,
                                                     int32_t n_lights, int32_t m, int32_t n,
                                                     const int32_t *__restrict__ pt_ids,
                                                     const int32_t *__restrict__ cl_ids, float r_min2, float eps,
                                                     float *__restrict__ out) {
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (g >= (int64_t)m * n) return;
    const int i = (int)(g / n), j = (int)(g % n);
    const int c = clamp_index(cl_ids[j], n_lights);
    const size_t N = (size_t)n_lights;
    const Light L = {{lights[c], lights[N + c], lights[2 * N + c]},
                     {lights[3 * N + c], lights[4 * N + c], lights[5 * N + c]},
                     lights[6 * N + c], lights[7 * N + c], lights[8 * N + c]};
    const PointData q = load_point(pts, pt_ids[i]);
    float o0, o1, o2;
    shade<KIND>(bvh, q, L, r_min2, eps, o0, o1, o2);
    out[3 * g] = o0;
    out[3 * g + 1] = o1;
    out[3 * g + 2] = o2;
}

template <int KIND>
__global__ __launch_bounds__(256) void k_eval_pairs(Bvh bvh, vplmc_points pts, vplmc_lights l, int64_t n,
                                                    const int32_t *__restrict__ pid,
                                                    const int32_t *__restrict__ lid, float r_min2, float eps,
                                                    float *__restrict__ out) {
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (g >= n) return;
    const int c = clamp_index(lid[g], l.n);
    const Light L = {{l.x[c], l.y[c], l.z[c]}, {l.nx[c], l.ny[c], l.nz[c]}, l.ir[c], l.ig[c], l.ib[c]};
    const PointData q = load_point(pts, pid[g]);
    float o0, o1, o2;
    shade<KIND>(bvh, q, L, r_min2, eps, o0, o1, o2);
    out[3 * g] = o0;
    out[3 * g + 1] = o1;
    out[3 * g + 2] = o2;
}

// Brute-force column sum against triangles, or against few spheres: one thread per point and light chunk (grid.y),
// lights staged through LDS; FP32 entries summed in FP64, chunk partial sums
// added to the zeroed output with FP64 atomics.  Bound by the shadow rays'
// traversal, whose latency needs wavefronts: the chunk (BF_MIN_CHUNK to
// BF_CHUNK lights) is the largest that still gives BF_GRID_PER_CU workgroups
// per CU (163,842 triangles, 1,024 points, 512 lights: chunks of 64 5.2 ms, of 16 1.4).
constexpr int BF_TILE = 256;
constexpr int BF_CHUNK = 2048, BF_MIN_CHUNK = 16;
constexpr int BF_GRID_PER_CU = 16;
// Spheres so few, or spheres times lights so few, that ordering the points and
// listing the spheres costs more than it saves (a call with one light 23 us here,
// 50-70 in k_brute_spheres).  us here / there, 1,024 points: 4 spheres 56 / 108
// (16 lights), 212 / 316 (16,384); 32 spheres 41 / 74 (4), 92 / 117 (16), 364 / 358
// (16,384); 128 spheres 77 / 85 (4), 230 / 164 (16); 512 spheres 54 / 86 (1), 133 /
// 133 (4).  8,192 points and 16,384 lights: 8 spheres 1,320 / 1,572, 12 spheres
// 1,728 / 1,536.
constexpr int BF_FEW_SPHERES = 8;
constexpr int64_t BF_FEW_TESTS = 512;
template <int KIND>
__global__ __launch_bounds__(256) void k_brute_force(Bvh bvh, vplmc_points pts, vplmc_lights l, int32_t n_out,
                                                     const int32_t *__restrict__ pid, int32_t chunk, float r_min2,
                                                     float eps, double *__restrict__ out) {
    __shared__ float sl[9][BF_TILE];
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    const bool active = g < n_out;
    PointData q{};
    if (active) q = load_point(pts, pid ? pid[g] : g);
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    const int c0 = blockIdx.y * chunk;
    const int c1 = min(l.n, c0 + chunk);
    for (int b = c0; b < c1; b += BF_TILE) {
        const int c = b + threadIdx.x;
        if (c < c1) {
            sl[0][threadIdx.x] = l.x[c];
            sl[1][threadIdx.x] = l.y[c];
            sl[2][threadIdx.x] = l.z[c];
            sl[3][threadIdx.x] = l.nx[c];
            sl[4][threadIdx.x] = l.ny[c];
            sl[5][threadIdx.x] = l.nz[c];
            sl[6][threadIdx.x] = l.ir[c];
            sl[7][threadIdx.x] = l.ig[c];
            sl[8][threadIdx.x] = l.ib[c];
        }
        __syncthreads();
        const int cnt = min(BF_TILE, c1 - b);
        if (active) {
            for (int k = 0; k < cnt; ++k) {
                const Light L = {{sl[0][k], sl[1][k], sl[2][k]}, {sl[3][k], sl[4][k], sl[5][k]}, sl[6][k], sl[7][k],
                                 sl[8][k]};
                float o0, o1, o2;
                shade<KIND>(bvh, q, L, r_min2, eps, o0, o1, o2);
                a0 += (double)o0;
                a1 += (double)o1;
                a2 += (double)o2;
            }
        }
        __syncthreads();
    }
    if (active) {
        atomicAdd(out + 3 * (size_t)g, a0);
        atomicAdd(out + 3 * (size_t)g + 1, a1);
        atomicAdd(out + 3 * (size_t)g + 2, a2);
    }
}

// Brute-force column sum against spheres.  A workgroup takes a segment of BS_SEG
// consecutive outputs, orders its points along a Morton curve over their two
// longest axes (a bitonic sort in LDS, the same in every workgroup of the segment;
// the order decides only which points share a wavefront), and its wavefronts each take 64 neighbours of that order and one
// light after another, so that the 64 shadow segments lie in one narrow shaft
// whose spheres are listed once (shaft_list).  With fewer runs of 64 points than
// wavefronts, several wavefronts share a run and split its lights.  FP32 entries
// summed in FP64, partial sums added to the zeroed output with FP64 atomics.
// Bound by VALU issue (0.80 busy) once the latency of listing (several dependent
// loads per list) is covered, hence 8 wavefronts per SIMD although some registers
// spill: 5.3 ms against 5.9 without.  8,192 points against 16,384 lights and 512 spheres 14.7 ->
// 5.1 ms (with a traversal per ray, points in caller order), 64 points 1.47 ->
// 0.44 ms, 16 spheres and 4,096 lights 0.84 -> 0.53 ms, 65,536 small spheres 15.4
// -> 10.1 ms.  BS_GRID_PER_CU workgroups per CU even out the ends (4: 6.0 ms,
// 16: as 8); each orders its segment again.
constexpr int BS_SEG = 4096, BS_THREADS = 1024, BS_WAVES = BS_THREADS / 64;
constexpr int BS_AXIS = 64;                  // Morton cells per axis
constexpr int BS_GRID_PER_CU = 8, BS_MIN_CHUNK = 64;

__device__ __forceinline__ uint32_t spread6(uint32_t x) {        // bit b of x to bit 2 b
    x = (x | (x << 4)) & 0x30Fu;
    x = (x | (x << 2)) & 0x333u;
    return (x | (x << 1)) & 0x555u;
}

__global__ __launch_bounds__(BS_THREADS) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_brute_spheres(
    Bvh bvh, vplmc_points pts, vplmc_lights l, int32_t n_out, const int32_t *__restrict__ pid, int32_t chunk, float r_min2,
    float eps, double *__restrict__ out) {
    __shared__ float4 lists[BS_WAVES][SHAFT_CAP];
    __shared__ uint32_t order[BS_SEG];       // Morton cell << 12 | output of the segment
    __shared__ float ext[BS_WAVES][6];
    constexpr int PER_SEG = BS_SEG / (64 * BS_WAVES);            // workgroups of a full segment
    constexpr int PER_THREAD = BS_SEG / BS_THREADS;
    static_assert(BS_SEG <= 4096 && BS_AXIS == 64, "12 bits each");
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int base = blockIdx.x / PER_SEG * BS_SEG;
    const int len = min(BS_SEG, n_out - base);
    const int run0 = blockIdx.x % PER_SEG * BS_WAVES;            // first run of 64 points
    const int runs = min(BS_WAVES, (len + 63) / 64 - run0);
    // positions, their box, the two longest axes
    float x[PER_THREAD][3], lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) lo[a] = hi[a] = INFINITY;        // hi: minimum of the negated
#pragma unroll
    for (int u = 0; u < PER_THREAD; ++u) {
        const int i = min(t + u * BS_THREADS, len - 1);
        const int p = clamp_index(pid ? pid[base + i] : base + i, pts.m);
        x[u][0] = pts.px[p];
        x[u][1] = pts.py[p];
        x[u][2] = pts.pz[p];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = fminf(lo[a], x[u][a]);
            hi[a] = fminf(hi[a], -x[u][a]);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = wave_min(lo[a]);
        hi[a] = wave_min(hi[a]);
        if (lane == 0) {
            ext[w][a] = lo[a];
            ext[w][3 + a] = hi[a];
        }
    }
    __syncthreads();
    float len3[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = hi[a] = INFINITY;
        for (int v = 0; v < BS_WAVES; ++v) {
            lo[a] = fminf(lo[a], ext[v][a]);
            hi[a] = fminf(hi[a], ext[v][3 + a]);
        }
        len3[a] = -hi[a] - lo[a];
    }
    const int drop = len3[0] < len3[1] ? (len3[0] < len3[2] ? 0 : 2) : (len3[1] < len3[2] ? 1 : 2);
#pragma unroll
    for (int u = 0; u < PER_THREAD; ++u) {
        uint32_t c[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {      // (not a number, as from an empty or infinite box: cell 0)
            const float f = (x[u][a] - lo[a]) / len3[a] * (float)BS_AXIS;
            c[a] = (uint32_t)fminf(fmaxf(f, 0.0f), (float)(BS_AXIS - 1));
        }
        const uint32_t key = spread6(drop == 0 ? c[1] : c[0]) | spread6(drop == 2 ? c[1] : c[2]) << 1;
        const int i = t + u * BS_THREADS;
        order[i] = i < len ? key << 12 | (uint32_t)i : 0xFFFFFFFFu;
    }
    __syncthreads();
    for (int k = 2; k <= BS_SEG; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
            for (int u = 0; u < PER_THREAD / 2; ++u) {
                const int e = t + u * BS_THREADS;                // compare-exchange e of the step
                const int i = (e & ~(j - 1)) << 1 | (e & (j - 1));
                const uint32_t a = order[i], b = order[i | j];
                if ((a > b) == ((i & k) == 0)) {
                    order[i] = b;
                    order[i | j] = a;
                }
            }
            __syncthreads();
        }
    // the wavefront's run of points and its share of the chunk's lights
    int slots = 1;
    while (slots < runs) slots *= 2;
    const int run = w & (slots - 1), split = BS_WAVES / slots, part = w / slots;
    if (run >= runs) return;
    const int i = (run0 + run) * 64 + lane;
    const bool active = i < len;
    const int g = base + (active ? (int)(order[i] & 4095u) : 0);
    PointData q{};
    if (active) q = load_point(pts, pid ? pid[g] : g);
    const P3 o = {fmaf(eps, q.n.x, q.x.x), fmaf(eps, q.n.y, q.x.y), fmaf(eps, q.n.z, q.x.z)};
    const float of[3] = {o.x, o.y, o.z};
    float alo[3], ahi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        alo[a] = wave_min(active ? of[a] : INFINITY);
        ahi[a] = -wave_min(active ? -of[a] : INFINITY);
    }
    // origins beyond any box, or too many groups: the traversal for every light
    const bool shaft = bvh.n_groups <= SHAFT_MAX_GROUPS && __ballot(active && !boxed(o)) == 0;
    int over = 0;                          // lists that overflowed, less those that did not
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    const int c1 = min(l.n, (int)(blockIdx.y + 1) * chunk);
    for (int c = blockIdx.y * chunk + part; c < c1; c += split) {
        const Light L = {{l.x[c], l.y[c], l.z[c]}, {l.nx[c], l.ny[c], l.nz[c]}, l.ir[c], l.ig[c], l.ib[c]};
        float o0 = 0.f, o1 = 0.f, o2 = 0.f;
        bool ray = false;
        if (active) ray = entry_unoccluded(q, L, r_min2, o0, o1, o2);
        if (__ballot(ray) == 0) continue;
        bool occ = false;
        int count = SHAFT_CAP + 1;
        if (shaft && over <= 4) {
            float blo[3] = {L.y.x, L.y.y, L.y.z}, bhi[3] = {L.y.x, L.y.y, L.y.z};
            float al[3] = {alo[0], alo[1], alo[2]}, ah[3] = {ahi[0], ahi[1], ahi[2]};
            count = bvh.n_groups ? shaft_list(bvh, lists[w], al, ah, blo, bhi) : 0;
            over = count > SHAFT_CAP ? over + 1 : max(over - 1, 0);
        }
        if (count <= SHAFT_CAP)
            occ = list_occluded(lists[w], count, ray, o, L.y);
        else if (ray)
            occ = occluded_in(BvhGlobal<0>{bvh}, bvh.n_nodes, o, sub(L.y, o));
        if (ray && !occ) {
            a0 += (double)o0;
            a1 += (double)o1;
            a2 += (double)o2;
        }
    }
    if (active) {
        atomicAdd(out + 3 * (size_t)g, a0);
        atomicAdd(out + 3 * (size_t)g + 1, a1);
        atomicAdd(out + 3 * (size_t)g + 2, a2);
    }
}

// workgroups of a chunk of lights: whole segments, then the last one's runs
int64_t bs_blocks(int32_t n_out) {
    const int64_t per_seg = BS_SEG / (64 * BS_WAVES);
    return n_out / BS_SEG * per_seg + (n_out % BS_SEG + 64 * BS_WAVES - 1) / (64 * BS_WAVES);
}

__global__ void k_zero_f64(double *p, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

// Training targets of the learned proposal from fully evaluated slices: per
// (slice, column) the mean and mean square of t = R + G + B over every row
// (one thread per column, FP64 sums in row order), then per slice
// p*_j ~ sigma_j + PROPOSAL_TARGET_MIX mean(sigma) (mix 3).
template <int KIND>
__global__ __launch_bounds__(256) void k_target_moments(Bvh bvh, vplmc_points pts, const float *__restrict__ lights,
                                                        int32_t n_lights, const SliceDesc *__restrict__ desc, int S,
                                                        int64_t total_cols, const int32_t *__restrict__ pt_ids,
                                                        const int32_t *__restrict__ cl_ids, float r_min2, float eps,
                                                        double *__restrict__ m1, double *__restrict__ m2) {
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (g >= total_cols) return;
    int lo = 0, hi = S;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (desc[mid].off_colptr - mid <= g) lo = mid; else hi = mid;
    }
    const int s = lo;
    const SliceDesc d = desc[s];
    const int64_t j = g - (d.off_colptr - s);
    const int c = clamp_index(cl_ids[d.cl_off + j], n_lights);
    const size_t N = (size_t)n_lights;
    const Light L = {{lights[c], lights[N + c], lights[2 * N + c]},
                     {lights[3 * N + c], lights[4 * N + c], lights[5 * N + c]},
                     lights[6 * N + c], lights[7 * N + c], lights[8 * N + c]};
    double s1 = 0.0, s2 = 0.0;
    for (int i = 0; i < d.m; ++i) {
        const PointData q = load_point(pts, pt_ids[d.pt_off + i]);
        float o0, o1, o2;
        shade<KIND>(bvh, q, L, r_min2, eps, o0, o1, o2);
        const double tv = (double)((o0 + o1) + o2);
        s1 += tv;
        s2 += tv * tv;
    }
    m1[d.off_col + j] = s1 / d.m;
    m2[d.off_col + j] = s2 / d.m;
}

__global__ __launch_bounds__(256) void k_target_norm(const SliceDesc *__restrict__ desc, const double *__restrict__ m1,
                                                     const double *__restrict__ m2, float *__restrict__ pstar) {
    __shared__ double red[256];
    const int s = blockIdx.x, t = threadIdx.x;
    const SliceDesc d = desc[s];
    double a = 0.0;
    for (int j = t; j < d.n; j += 256) {
        const int64_t o = d.off_col + j;
        a += sqrt(fmax(0.0, m2[o] - m1[o] * m1[o]));
    }
    red[t] = a;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (t < w) red[t] += red[t + w];
        __syncthreads();
    }
    const double mean = red[0] / d.n;
    const double add = PROPOSAL_TARGET_MIX * (mean > 0.0 ? mean : 1.0);
    const double total = red[0] + add * d.n;
    for (int j = t; j < d.n; j += 256) {
        const int64_t o = d.off_col + j;
        pstar[o] = (float)((sqrt(fmax(0.0, m2[o] - m1[o] * m1[o])) + add) / total);
    }
}

unsigned blocks_for(int64_t n, int threads) { return (unsigned)((n + threads - 1) / threads); }

}  // namespace

int launch_targets(hipStream_t st, const vplmc_plan &plan, const SliceDesc *desc, const Bvh &bvh,
                   const vplmc_points &pts, const float *lights, int32_t n_lights, const int32_t *pt_ids,
                   const int32_t *cl_ids, const vplmc_params &prm, double *moments, float *pstar) {
    if (plan.n_slices <= 0) return VPLMC_OK;
    const int64_t cols = plan.tot_col;
    if (bvh.kind == 1)
        hipLaunchKernelGGL((k_target_moments<1>), dim3(blocks_for(cols, 256)), dim3(256), 0, st, bvh, pts, lights, n_lights,
                           desc, plan.n_slices, cols, pt_ids, cl_ids, prm.r_min * prm.r_min, prm.ray_eps, moments,
                           moments + cols);
    else
        hipLaunchKernelGGL((k_target_moments<0>), dim3(blocks_for(cols, 256)), dim3(256), 0, st, bvh, pts, lights, n_lights,
                           desc, plan.n_slices, cols, pt_ids, cl_ids, prm.r_min * prm.r_min, prm.ray_eps, moments,
                           moments + cols);
    VPLMC_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_target_norm, dim3(plan.n_slices), dim3(256), 0, st, desc, moments, moments + cols, pstar);
    VPLMC_HIP(hipGetLastError());
    return VPLMC_OK;
}

int launch_eval_omega(hipStream_t st, const Bvh &bvh, const vplmc_points &pts, const float *lights,
                      int32_t n_lights, const SliceDesc *desc, int32_t n_slices, const int32_t *pt_ids,
                      const int32_t *cl_ids, const uint32_t *keys, int64_t n_keys, int which,
                      const int32_t *stats, const vplmc_params &prm, float *vals, int threads, int n_cu,
                      unsigned long long *rays) {
    if (n_keys <= 0) return VPLMC_OK;
    if (threads != 64 && threads != 128 && threads != 256) threads = 256;   // __launch_bounds__(256)
    // enough workgroups to fill the chip several times over; each walks the
    // samples with a grid stride
    const int64_t blocks = std::min<int64_t>(blocks_for(n_keys, threads), (int64_t)EVAL_GRID_PER_CU * n_cu);
    const size_t staged = ((size_t)2 * bvh.n_nodes + bvh.n_spheres) * sizeof(float4);
    if (bvh.n_nodes > 0 && staged <= (size_t)EVAL_LDS_BYTES) {
        if (bvh.kind == 1)
            hipLaunchKernelGGL((k_eval_omega<true, 1>), dim3((unsigned)blocks), dim3(threads), staged, st, bvh, pts, lights,
                               n_lights, desc, n_slices, pt_ids, cl_ids, keys, n_keys, which, stats,
                               prm.r_min * prm.r_min, prm.ray_eps, vals, rays);
        else
            hipLaunchKernelGGL((k_eval_omega<true, 0>), dim3((unsigned)blocks), dim3(threads), staged, st, bvh, pts, lights,
                               n_lights, desc, n_slices, pt_ids, cl_ids, keys, n_keys, which, stats,
                               prm.r_min * prm.r_min, prm.ray_eps, vals, rays);
    } else {
        if (bvh.kind == 1)
            hipLaunchKernelGGL((k_eval_omega<false, 1>), dim3((unsigned)blocks), dim3(threads), 0, st, bvh, pts, lights,
                               n_lights, desc, n_slices, pt_ids, cl_ids, keys, n_keys, which, stats,
                               prm.r_min * prm.r_min, prm.ray_eps, vals, rays);
        else
            hipLaunchKernelGGL((k_eval_omega<false, 0>), dim3((unsigned)blocks), dim3(threads), 0, st, bvh, pts, lights,
                               n_lights, desc, n_slices, pt_ids, cl_ids, keys, n_keys, which, stats,
                               prm.r_min * prm.r_min, prm.ray_eps, vals, rays);
    }
    VPLMC_HIP(hipGetLastError());
    return VPLMC_OK;
}

template <bool STAGED, int KIND>
static int coarsen_eps(hipStream_t st, const vplmc_plan &plan, const Bvh &bvh, size_t staged, const vplmc_points &pts,
                       const float *lights, const SliceDesc *desc, const int32_t *pt_ids, CoarsenTree tr,
                       const CoarsenSlices &cs, const vplmc_params &prm, int n_cu, unsigned long long *counts) {
    const int threads = 256;
    const float r_min2 = prm.r_min * prm.r_min;
    if (bvh.n_nodes == 0) tr.n_front = 1;        // without shadow rays an entry costs no more than its look-up
    const bool table = tr.n_front > 1;
    const size_t runs = table ? plan.top_runs.size() - 1 : 1;
    for (size_t k = 0; k < runs; ++k) {
        const int32_t s0 = table ? plan.top_runs[k] : 0, s1 = table ? plan.top_runs[k + 1] : plan.n_slices;
        const int64_t row0 = plan.desc[s0].off_row - s0;
        if (table) {
            const int64_t rows = plan.desc[s1 - 1].off_row - (s1 - 1) + plan.desc[s1 - 1].m - row0;
            hipLaunchKernelGGL((k_coarsen_top<STAGED, KIND>),
                               dim3(blocks_for(rows, threads), (unsigned)((tr.n_front + TOP_LIGHTS - 1) / TOP_LIGHTS)),
                               dim3(threads), staged, st, bvh, pts, lights, desc, s0, s1, row0, rows,
                               (int64_t)plan.pixels, pt_ids, tr, cs, r_min2, prm.ray_eps);
            VPLMC_HIP(hipGetLastError());
        }
        const int64_t total = (int64_t)(s1 - s0) * plan.pixels;
        const int64_t blocks = std::min<int64_t>(blocks_for(total, threads), (int64_t)EVAL_GRID_PER_CU * n_cu);
        hipLaunchKernelGGL((k_coarsen_eps<STAGED, KIND>), dim3((unsigned)blocks), dim3(threads), staged, st, bvh, pts,
                           lights, desc, s0, row0, total, (int64_t)plan.pixels, pt_ids, tr, cs, prm.seed, r_min2,
                           prm.ray_eps, counts);
        VPLMC_HIP(hipGetLastError());
    }
    return VPLMC_OK;
}

// Draws of a launch (over all slices) from which the level-by-level walk pays:
// with fewer its longer chain of loads per level costs more than the shared lists
// save.  Merge-error phase, ms, own walk per thread / level by level: 2.6e5 draws
// 0.52 / 0.62 (512 spheres, 4,096 leaves) and 0.97 / 0.69 (2,048, 16,384), 5.2e5
// 0.84 / 0.80 and 1.19 / 0.61, 2.1e6 2.54 / 1.49 and 3.81 / 1.54; triangles 6.6e4
// 0.84 / 1.07, 1.0e6 4.4 / 4.0.  Dense occluders whose lists overflow lose up to
// a quarter of it at 1e6 draws (1.06 / 1.40 ms) and nothing at 8e6 (6.3 / 6.2).
// Without occluders there is nothing to share: 2.1e6 0.81 / 0.95, 8.4e6 2.65 / 2.31.
constexpr int64_t COARSEN_LEVELS_FROM = 1 << 19;
constexpr int64_t COARSEN_LEVELS_FROM_NO_OCCLUDERS = 1 << 22;

int launch_coarsen_eps(hipStream_t st, const vplmc_plan &plan, const Bvh &bvh, const vplmc_points &pts,
                       const float *lights, const SliceDesc *desc, const int32_t *pt_ids, const CoarsenTree &tr,
                       const CoarsenSlices &cs, const vplmc_params &prm, int n_cu, unsigned long long *counts) {
    if (plan.n_slices <= 0 || plan.pixels <= 0) return VPLMC_OK;
    const size_t staged = ((size_t)2 * bvh.n_nodes + bvh.n_spheres) * sizeof(float4);
    const bool fits = bvh.n_nodes > 0 && staged <= (size_t)EVAL_LDS_BYTES;
    const int64_t total = (int64_t)plan.n_slices * plan.pixels;
    if (total < (bvh.n_nodes > 0 ? COARSEN_LEVELS_FROM : COARSEN_LEVELS_FROM_NO_OCCLUDERS)) {
        const int threads = 256;
        const int64_t blocks = std::min<int64_t>(blocks_for(total, threads), (int64_t)EVAL_GRID_PER_CU * n_cu);
        auto walk = bvh.kind == 1 ? (fits ? k_coarsen_walk<true, 1> : k_coarsen_walk<false, 1>)
                                  : (fits ? k_coarsen_walk<true, 0> : k_coarsen_walk<false, 0>);
        hipLaunchKernelGGL(walk, dim3((unsigned)blocks), dim3(threads), fits ? staged : 0, st, bvh, pts, lights, desc,
                           total, (int64_t)plan.pixels, pt_ids, tr, cs, prm.seed, prm.r_min * prm.r_min, prm.ray_eps,
                           counts);
        VPLMC_HIP(hipGetLastError());
        return VPLMC_OK;
    }
    const bool stage = bvh.kind == 1 && fits;   // spheres: occluded_shaft
    auto run = stage ? coarsen_eps<true, 1> : (bvh.kind == 1 ? coarsen_eps<false, 1> : coarsen_eps<false, 0>);
    return run(st, plan, bvh, stage ? staged : 0, pts, lights, desc, pt_ids, tr, cs, prm, n_cu, counts);
}

int launch_full_matrix(hipStream_t st, const Bvh &bvh, const vplmc_points &pts, const float *lights,
                       int32_t n_lights, int32_t m, int32_t n, const int32_t *pt_ids, const int32_t *cl_ids,
                       const vplmc_params &prm, float *out) {
    const int64_t total = (int64_t)m * n;
    if (total <= 0) return VPLMC_OK;
    if (bvh.kind == 1)
        hipLaunchKernelGGL((k_full_matrix<1>), dim3(blocks_for(total, 256)), dim3(256), 0, st, bvh, pts, lights, n_lights, m, n,
                           pt_ids, cl_ids, prm.r_min * prm.r_min, prm.ray_eps, out);
    else
        hipLaunchKernelGGL((k_full_matrix<0>), dim3(blocks_for(total, 256)), dim3(256), 0, st, bvh, pts, lights, n_lights, m, n,
                           pt_ids, cl_ids, prm.r_min * prm.r_min, prm.ray_eps, out);
    VPLMC_HIP(hipGetLastError());
    return VPLMC_OK;
}

int launch_eval_pairs(hipStream_t st, const Bvh &bvh, const vplmc_points &pts, const vplmc_lights &l, int64_t n,
                      const int32_t *pid, const int32_t *lid, const vplmc_params &prm, float *out) {
    if (n <= 0) return VPLMC_OK;
    if (bvh.kind == 1)
        hipLaunchKernelGGL((k_eval_pairs<1>), dim3(blocks_for(n, 256)), dim3(256), 0, st, bvh, pts, l, n, pid, lid,
                           prm.r_min * prm.r_min, prm.ray_eps, out);
    else
        hipLaunchKernelGGL((k_eval_pairs<0>), dim3(blocks_for(n, 256)), dim3(256), 0, st, bvh, pts, l, n, pid, lid,
                           prm.r_min * prm.r_min, prm.ray_eps, out);
    VPLMC_HIP(hipGetLastError());
    return VPLMC_OK;
}

int launch_brute_force(hipStream_t st, const Bvh &bvh, const vplmc_points &pts, const vplmc_lights &l,
                       int32_t n_out, const int32_t *pid, const vplmc_params &prm, int n_cu, double *out) {
    if (n_out <= 0) return VPLMC_OK;
    const size_t nz = 3 * (size_t)n_out;
    hipLaunchKernelGGL(k_zero_f64, dim3((unsigned)std::min<size_t>((nz + 255) / 256, 65536)), dim3(256), 0, st, out, nz);
    VPLMC_HIP(hipGetLastError());
    if (l.n <= 0) return VPLMC_OK;
    const bool plain = bvh.kind == 1 || bvh.n_spheres <= BF_FEW_SPHERES || (int64_t)bvh.n_spheres * l.n <= BF_FEW_TESTS;
    const int64_t blocks = plain ? blocks_for(n_out, 256) : bs_blocks(n_out);
    const int64_t want = (int64_t)(plain ? BF_GRID_PER_CU : BS_GRID_PER_CU) * n_cu;
    const int32_t smallest = plain ? BF_MIN_CHUNK : BS_MIN_CHUNK;
    int32_t chunk = BF_CHUNK;
    // (grid.y is at most 65,535)
    while (chunk > smallest && blocks * ((l.n + chunk - 1) / chunk) < want && l.n / (chunk / 2) < 65535) chunk /= 2;
    const unsigned chunks = (unsigned)((l.n + (int64_t)chunk - 1) / chunk);
    if (plain)
        hipLaunchKernelGGL((bvh.kind == 1 ? k_brute_force<1> : k_brute_force<0>), dim3((unsigned)blocks, chunks), dim3(256), 0, st, bvh, pts, l, n_out,
                           pid, chunk, prm.r_min * prm.r_min, prm.ray_eps, out);
    else
        hipLaunchKernelGGL(k_brute_spheres, dim3((unsigned)blocks, chunks), dim3(BS_THREADS), 0, st, bvh, pts, l, n_out,
                           pid, chunk, prm.r_min * prm.r_min, prm.ray_eps, out);
    VPLMC_HIP(hipGetLastError());
    return VPLMC_OK;
}

}  // namespace vplmc
