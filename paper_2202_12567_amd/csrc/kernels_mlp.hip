// Learned second-pass proposal: per-(slice, column) features from the first
// pass, a 12 -> 128 -> 128 -> 1 GELU network predicting the log of a column
// sampling density, its training (softmax-KL loss, backward, Adam) and the
// training targets from fully evaluated slices.  The paper samples columns by
// g(j) = max C_j - min C_j because columns whose results vary are important
// (Sec. 5) and names image-space-guided sampling as future work (Sec. 7);
// the network estimates that importance from the same sparse observations.
//
// Weights are used rounded to bfloat16 (round to nearest even) and the two
// hidden activations are rounded to bfloat16; accumulation is FP32.  The
// 128 x 128 layer of inference runs on MFMA (v_mfma_f32_32x32x8 bf16): one
// wavefront owns 32 rows, computes their layer-1 activations directly in
// the MFMA A-operand layout, and reduces the output layer across lanes.
// Training has the same rounding points (its kernels' comment says how it runs).

#include <algorithm>
#include <type_traits>

#include "vplmc_internal.h"

namespace vplmc {
namespace {

constexpr int WAVE = 64;
constexpr float SQRT_2_OVER_PI = 0.7978845608028654f;

// parameter offsets in the flat FP32 vector (W1 b1 W2 b2 W3 b3)
constexpr int P_W1 = 0;
constexpr int P_B1 = P_W1 + MLP_HID * MLP_IN;
constexpr int P_W2 = P_B1 + MLP_HID;
constexpr int P_B2 = P_W2 + MLP_HID * MLP_HID;
constexpr int P_W3 = P_B2 + MLP_HID;
constexpr int P_B3 = P_W3 + MLP_HID;

__device__ __forceinline__ float bf16r(float x) {
    uint32_t u = __float_as_uint(x);
    u = (u + 0x7FFFu + ((u >> 16) & 1u)) & 0xFFFF0000u;
    return __uint_as_float(u);
}
__device__ __forceinline__ uint16_t bf16bits(float x) { return (uint16_t)(__float_as_uint(bf16r(x)) >> 16); }

__device__ __forceinline__ float gelu(float x) {
    return 0.5f * x * (1.0f + tanhf(SQRT_2_OVER_PI * (x + 0.044715f * x * x * x)));
}

// LDS written by some lanes of a wavefront and then read by others
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// features: one workgroup per slice
//   mu = first-pass mean of t; per column j:
//   0 log1p(mean/mu) 1 log1p(std/mu) 2 log1p((max-min)/mu) 3 count/(N1/n)
//   4 zero fraction 5 log1p(cluster bbox diag / dist) 6 log1p(dist / slice diag)
//   7 cos(slice mean normal, slice->cluster) 8 cos(cluster normal, cluster->slice)
//   9 log1p(I_c / mean I over the cut) 10 log(members) 11 1 - |slice mean normal|
// Member counts come from the cut's offsets, or (light coarsening: columns
// are tree nodes) from node_members.
__global__ __launch_bounds__(256) void k_features(const SliceDesc *__restrict__ desc, vplmc_points pts,
                                                  const int32_t *__restrict__ pt_ids,
                                                  const int32_t *__restrict__ cl_ids, const float *__restrict__ lights,
                                                  int32_t nc, const float *__restrict__ bbox, vplmc_cut cut,
                                                  const int32_t *__restrict__ node_members,
                                                  const int32_t *__restrict__ cnt, const float *__restrict__ mn,
                                                  const float *__restrict__ mx, const double *__restrict__ sum,
                                                  const double *__restrict__ sumsq, const int32_t *__restrict__ zeros,
                                                  float *__restrict__ geo_out, float *__restrict__ F) {
    __shared__ double red[8][256];
    __shared__ float geo[8];
    __shared__ double mu_s, imean_s;
    const int s = blockIdx.x;
    const SliceDesc d = desc[s];
    const int t = threadIdx.x;
    const size_t N = (size_t)nc;
    // slice geometry and first-pass mean, fixed-order reductions
    double a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int i = t; i < d.m; i += 256) {
        const int p = clamp_index(pt_ids[d.pt_off + i], pts.m);
        const float x = pts.px[p], y = pts.py[p], z = pts.pz[p];
        a[0] += x; a[1] += y; a[2] += z;
        a[3] += pts.nx[p]; a[4] += pts.ny[p]; a[5] += pts.nz[p];
        lo[0] = fminf(lo[0], x); lo[1] = fminf(lo[1], y); lo[2] = fminf(lo[2], z);
        hi[0] = fmaxf(hi[0], x); hi[1] = fmaxf(hi[1], y); hi[2] = fmaxf(hi[2], z);
    }
    for (int j = t; j < d.n; j += 256) {
        a[6] += sum[d.off_col + j];
        const int c = clamp_index(cl_ids[d.cl_off + j], nc);
        a[7] += (double)((lights[6 * N + c] + lights[7 * N + c]) + lights[8 * N + c]);
    }
    for (int k = 0; k < 8; ++k) red[k][t] = a[k];
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (t < w)
            for (int k = 0; k < 8; ++k) red[k][t] += red[k][t + w];
        __syncthreads();
    }
    // bbox: reuse the reduction for min / max (as doubles)
    double bl[3] = {lo[0], lo[1], lo[2]}, bh[3] = {hi[0], hi[1], hi[2]};
    double tot[8];
    for (int k = 0; k < 8; ++k) tot[k] = red[k][0];
    __syncthreads();
    for (int k = 0; k < 3; ++k) {
        red[k][t] = bl[k];
        red[3 + k][t] = bh[k];
    }
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (t < w)
            for (int k = 0; k < 3; ++k) {
                red[k][t] = fmin(red[k][t], red[k][t + w]);
                red[3 + k][t] = fmax(red[3 + k][t], red[3 + k][t + w]);
            }
        __syncthreads();
    }
    if (t == 0) {
        const double im = 1.0 / (double)d.m;
        const double dx = red[3][0] - red[0][0], dy = red[4][0] - red[1][0], dz = red[5][0] - red[2][0];
        geo[0] = (float)(tot[0] * im);
        geo[1] = (float)(tot[1] * im);
        geo[2] = (float)(tot[2] * im);
        geo[3] = (float)sqrt(dx * dx + dy * dy + dz * dz);
        geo[4] = (float)(tot[3] * im);
        geo[5] = (float)(tot[4] * im);
        geo[6] = (float)(tot[5] * im);
        geo[7] = 0.f;
        const double mu = tot[6] / (double)(d.N1 > 0 ? d.N1 : 1);
        mu_s = mu > 0.0 ? mu : 1e-30;
        imean_s = tot[7] / (double)d.n;
        for (int k = 0; k < 8; ++k) geo_out[8 * s + k] = geo[k];
    }
    __syncthreads();
    const float cx = geo[0], cy = geo[1], cz = geo[2];
    const float diag = geo[3] + 1e-6f;
    const float mnx = geo[4], mny = geo[5], mnz = geo[6];
    const float nn = sqrtf(mnx * mnx + mny * mny + mnz * mnz) + 1e-12f;
    const double mu = mu_s;
    const float per = (float)d.N1 / (float)d.n;
    for (int j = t; j < d.n; j += 256) {
        const int64_t o = d.off_col + j;
        const int c = clamp_index(cl_ids[d.cl_off + j], nc);
        const float k = (float)cnt[o];
        const float safe = k > 0.f ? k : 1.f;
        const double mean = sum[o] / (double)safe;
        const double var = fmax(0.0, sumsq[o] / (double)safe - mean * mean);
        float *f = F + 12 * o;
        f[0] = (float)log1p(mean / mu);
        f[1] = (float)log1p(sqrt(var) / mu);
        f[2] = (float)log1p((double)(k > 0.f ? mx[o] - mn[o] : 0.f) / mu);
        f[3] = k / (per > 0.f ? per : 1.f);
        f[4] = k > 0.f ? (float)zeros[o] / safe : 0.f;
        const float px = lights[c] - cx, py = lights[N + c] - cy, pz = lights[2 * N + c] - cz;
        const float dist = sqrtf(px * px + py * py + pz * pz) + 1e-6f;
        const float ux = px / dist, uy = py / dist, uz = pz / dist;
        const float bx = bbox[3 * N + c] - bbox[c], by = bbox[4 * N + c] - bbox[N + c], bz = bbox[5 * N + c] - bbox[2 * N + c];
        f[5] = log1pf(sqrtf(bx * bx + by * by + bz * bz) / dist);
        f[6] = log1pf(dist / diag);
        f[7] = (ux * mnx + uy * mny + uz * mnz) / nn;
        f[8] = -(lights[3 * N + c] * ux + lights[4 * N + c] * uy + lights[5 * N + c] * uz);
        const double is = (double)((lights[6 * N + c] + lights[7 * N + c]) + lights[8 * N + c]);
        f[9] = (float)log1p(is / (imean_s + 1e-30));
        f[10] = logf((float)(node_members ? node_members[c] : cut.offsets[c + 1] - cut.offsets[c]));
        f[11] = 1.0f - nn;
    }
}

// ---------------------------------------------------------------------------
// inference: one wavefront = 32 rows; layer 2 on MFMA 32x32x8 bf16
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef float float16_t __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(256) void k_mlp_forward(const float *__restrict__ P, int64_t rows,
                                                     const float *__restrict__ F, float *__restrict__ y) {
    __shared__ float w1s[MLP_HID * MLP_IN];
    __shared__ float b1s[MLP_HID];
    __shared__ uint16_t w2s[MLP_HID * MLP_HID];   // bf16 bits, [h][k]
    __shared__ float b2s[MLP_HID], w3s[MLP_HID];
    const int t = threadIdx.x;
    for (int e = t; e < MLP_HID * MLP_IN; e += 256) w1s[e] = bf16r(P[P_W1 + e]);
    for (int e = t; e < MLP_HID; e += 256) {
        b1s[e] = P[P_B1 + e];
        b2s[e] = P[P_B2 + e];
        w3s[e] = bf16r(P[P_W3 + e]);
    }
    for (int e = t; e < MLP_HID * MLP_HID; e += 256) w2s[e] = bf16bits(P[P_W2 + e]);
    __syncthreads();
    const float b3 = P[P_B3];
    const int lane = t % WAVE, wave = t / WAVE;
    const int64_t r0 = ((int64_t)blockIdx.x * 4 + wave) * 32;
    if (r0 >= rows) return;
    const int i = lane % 32;          // A-operand row of this lane
    const int kh = lane / 32;         // which 4-wide k half of each 8-wide step
    const int64_t row = r0 + i;
    float f[MLP_IN];
#pragma unroll
    for (int q = 0; q < MLP_IN; ++q) f[q] = row < rows ? F[12 * row + q] : 0.f;
    // layer 1 in the A layout: step ks covers k = 8 ks + 4 kh + {0..3}
    short4_t A[16];
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
        short4_t v;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int k = 8 * ks + 4 * kh + c;
            float z = b1s[k];
#pragma unroll
            for (int q = 0; q < MLP_IN; ++q) z = fmaf(w1s[k * MLP_IN + q], f[q], z);
            v[c] = (short)bf16bits(gelu(z));
        }
        A[ks] = v;
    }
    // layer 2 (MFMA) and the output layer, four 32-column tiles of hidden units
    float part[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) part[v] = 0.f;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const int h = nt * 32 + (lane % 32);  // B-operand column / C column of this lane
        float16_t acc = {};
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) {
            short4_t b;
#pragma unroll
            for (int c = 0; c < 4; ++c) b[c] = (short)w2s[h * MLP_HID + 8 * ks + 4 * kh + c];
            acc = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(A[ks], b, acc, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float h2 = bf16r(gelu(acc[v] + b2s[h]));
            part[v] = fmaf(w3s[h], h2, part[v]);
        }
    }
    // sum over the 32 hidden-unit lanes of each half-wave
#pragma unroll
    for (int v = 0; v < 16; ++v) {
#pragma unroll
        for (int o = 16; o >= 1; o >>= 1) part[v] += __shfl_xor(part[v], o, WAVE);
    }
    if (lane % 32 == 0) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int r = (v / 4) * 8 + kh * 4 + (v % 4);   // C row of accumulator v
            if (r0 + r < rows) y[r0 + r] = part[v] + b3;
        }
    }
}

// ---------------------------------------------------------------------------
// training.  A wavefront owns 32 rows; lane l keeps row l % 32 through the
// whole network: of each 128-vector of hidden units it holds the 64 with
// index unit(t, v, l / 32), which is where a 32 x 32 MFMA result puts them
// (register v of tile t) and, the contraction order being free, where the next
// product's right operand takes them from, so no activation crosses lanes
// inside a pass.  The 128 x 128 products run on v_mfma_f32_32x32x16_bf16 with
// FP32 accumulation: forward both operands are bfloat16 anyway; backward
// dz2 (FP32) enters as three bfloat16 terms that sum to it exactly (its 24
// significant bits in eights), so every product is exact (the sums of W2^T dz2
// alone: relative RMS error 1.14e-7 against 64 bits, a chain of FP32 fmas 2.03e-7).  Nothing of the
// forward pass is kept: the backward pass recomputes it, which costs less
// than four 128-vectors of FP32 per row written and read back.  dW2 contracts
// over rows: the backward kernel leaves dz2 and h1 in the scratch and
// k_train_dw2 forms it with FP32 MFMA.  Each workgroup adds its partial
// gradients with FP32 atomics.
//
// Bound by the activations' VALU work (a sigmoid per hidden unit and pass; VALU
// 0.73 busy forward, 0.52 backward), dW2 by the matrix unit (0.35 busy) and its loads.
// Measured on one MI355X, 131,072 rows: forward 0.97 -> 0.053 ms, backward
// 5.53 -> 0.24 ms (0.161 and 0.076 for dW2), against FP32 VALU kernels that kept the activations in
// the scratch and added every 32-row block's gradients with 18,000 atomics.
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f4_t __attribute__((ext_vector_type(4)));

constexpr int TRAIN_ROWS = 32;            // rows of a wavefront
constexpr int TRAIN_FW = 4;               // wavefronts of a forward workgroup
constexpr int TRAIN_BW = 8;               // wavefronts of a backward workgroup
constexpr int TRAIN_W1 = 16;              // words per hidden unit of the staged first layer: 12 weights, bias, pad
constexpr int TRAIN_LD = 36;              // row stride of a wavefront's transposing tile (floats)

__device__ __forceinline__ int unit(int t, int v, int half) { return 32 * t + 8 * (v >> 2) + 4 * half + (v & 3); }

// W2 as the left operand of 32 x 32 x 16 products, in bfloat16: element
// ((4-tile * 8 + step) * 64 + lane) * 8 + c.  FORWARD: rows are output units
// h, contraction over input units k; else rows are k, contraction over h.
template <bool FORWARD>
__device__ void stage_w2(const float *__restrict__ P, uint16_t *w, int threads) {
    for (int e = threadIdx.x; e < MLP_HID * MLP_HID; e += threads) {
        const int h = e / MLP_HID, k = e % MLP_HID;
        const int row = FORWARD ? h : k, con = FORWARD ? k : h;
        const int half = (con >> 2) & 1, v = 4 * ((con % 32) >> 3) + (con & 3);
        const int step = 2 * (con / 32) + v / 8;
        w[(((row / 32) * 8 + step) * 64 + half * 32 + row % 32) * 8 + v % 8] = bf16bits(P[P_W2 + e]);
    }
}
__device__ void stage_w1(const float *__restrict__ P, float *w, int threads) {
    for (int e = threadIdx.x; e < MLP_HID * TRAIN_W1; e += threads) {
        const int k = e / TRAIN_W1, q = e % TRAIN_W1;
        w[e] = q < MLP_IN ? bf16r(P[P_W1 + k * MLP_IN + q]) : (q == MLP_IN ? P[P_B1 + k] : 0.f);
    }
}

// s = (1 + tanh(u)) / 2 = 1 / (1 + exp(-2 u)), u the GELU's argument at x;
// gelu = x s, gelu' = s + 2 x s (1 - s) u'(x).  s is kept as r + q, the
// reciprocal of d = fl(1 + e) and its correction for d's own rounding as well,
// and 1 - s is e s: 1 - s from a rounded s cancels where s is near 1.
// Past |2 u| = 80, s is 0 or 1 in FP32.  Relative RMS error of the slope on
// N(0, 1.5) 3.7e-8 (with 1 - s 1.55e-7, with tanhf 6.6e-8), of the activation
// 3.2e-8 (3.6e-8 with tanhf).
constexpr float LOG2_E = 1.44269504088896340736f, LOG2_E_LO = (float)(1.44269504088896340736 - (double)LOG2_E);
struct GeluSigmoid {
    float r, q, e, v;                     // s = r + q, e = exp(v), v = -2 u
};
__device__ __forceinline__ GeluSigmoid gelu_sigmoid(float x) {
    GeluSigmoid g;
    g.v = -2.0f * SQRT_2_OVER_PI * (x + 0.044715f * x * x * x);
    // exp of a value clamped to [-100, 80]: 2^n 2^f with n + f = v log2(e) as an unevaluated sum
    const float v = __builtin_amdgcn_fmed3f(g.v, -100.0f, 80.0f);
    const float hi = v * LOG2_E, lo = fmaf(v, LOG2_E_LO, fmaf(v, LOG2_E, -hi));
    const float n = rintf(hi);
    g.e = ldexpf(__builtin_amdgcn_exp2f((hi - n) + lo), (int)n);
    const float d = 1.0f + g.e;
    g.r = g.v > 80.0f ? 0.0f : __builtin_amdgcn_rcpf(d);
    g.q = fmaf(-(g.e - (d - 1.0f)), g.r, fmaf(-d, g.r, 1.0f)) * g.r;
    return g;
}
__device__ __forceinline__ float gelu_value(float x, const GeluSigmoid &g) {
    return fabsf(g.v) > 80.0f ? x * g.r : fmaf(x, g.r, x * g.q);     // (an infinite x times a correction of either sign)
}
__device__ __forceinline__ float gelu_slope(float x, const GeluSigmoid &g) {
    const float du = SQRT_2_OVER_PI * (1.0f + 3.0f * 0.044715f * x * x);
    const float s = g.r + g.q;
    const float slope = g.r + fmaf(2.0f * x * du, s * (g.e * s), g.q);
    return fabsf(g.v) > 80.0f ? s : slope;          // (x du may overflow there)
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {   // operands already representable
    return (__float_as_uint(lo) >> 16) | (__float_as_uint(hi) & 0xFFFF0000u);
}
// what the leading 8 significant bits leave of x (an infinity leaves nothing)
__device__ __forceinline__ float remainder_bf16(float x) {
    const float lead = __uint_as_float(__float_as_uint(x) & 0xFFFF0000u);
    return x == lead ? 0.f : x - lead;
}
__device__ __forceinline__ float16_t mfma_bf16(const uint4 &a, const uint4 &b, float16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c, 0, 0, 0);
}

// z1 of unit(t, v, half) of the lane's row
__device__ __forceinline__ float train_z1(const float (&f)[MLP_IN], const float *w1, int t, int v, int half) {
    const float4 *w = reinterpret_cast<const float4 *>(w1 + unit(t, v, half) * TRAIN_W1);
    const float4 u0 = w[0], u1 = w[1], u2 = w[2];
    float z = w[3].x;
    z = fmaf(u0.x, f[0], z);
    z = fmaf(u0.y, f[1], z);
    z = fmaf(u0.z, f[2], z);
    z = fmaf(u0.w, f[3], z);
    z = fmaf(u1.x, f[4], z);
    z = fmaf(u1.y, f[5], z);
    z = fmaf(u1.z, f[6], z);
    z = fmaf(u1.w, f[7], z);
    z = fmaf(u2.x, f[8], z);
    z = fmaf(u2.y, f[9], z);
    z = fmaf(u2.z, f[10], z);
    z = fmaf(u2.w, f[11], z);
    return z;
}

// layer 1 of the lane's row: h1 of step s (units of tile s / 2) as a right operand
__device__ __forceinline__ void train_layer1(const float (&f)[MLP_IN], const float *w1, int half, uint4 (&h1)[8]) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        uint32_t pk[8];
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
            float a[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float z = train_z1(f, w1, t, v + c, half);
                a[c] = bf16r(gelu_value(z, gelu_sigmoid(z)));
            }
            pk[v / 2] = pack_bf16(a[0], a[1]);
            __builtin_amdgcn_sched_barrier(0);     // bounds the staged weights in flight
        }
        h1[2 * t] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        h1[2 * t + 1] = make_uint4(pk[4], pk[5], pk[6], pk[7]);
    }
}

// z2 of the units of tile t
__device__ __forceinline__ float16_t train_layer2(const uint4 (&h1)[8], const uint4 *w2, const float *b2, int t, int lane) {
    float16_t z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = b2[unit(t, v, lane / 32)];
#pragma unroll
    for (int st = 0; st < 8; ++st) z = mfma_bf16(w2[(t * 8 + st) * 64 + lane], h1[st], z);
    return z;
}

__global__ __launch_bounds__(64 * TRAIN_FW) __attribute__((amdgpu_waves_per_eu(3))) void k_train_forward(const float *__restrict__ P, int64_t rows,
                                                                 const float *__restrict__ F, float *__restrict__ y) {
    constexpr int NT = 64 * TRAIN_FW;
    __shared__ __align__(16) uint16_t w2s[MLP_HID * MLP_HID];
    __shared__ __align__(16) float w1s[MLP_HID * TRAIN_W1];
    __shared__ float b2s[MLP_HID], w3s[MLP_HID];
    stage_w2<true>(P, w2s, NT);
    stage_w1(P, w1s, NT);
    for (int e = threadIdx.x; e < MLP_HID; e += NT) {
        b2s[e] = P[P_B2 + e];
        w3s[e] = bf16r(P[P_W3 + e]);
    }
    __syncthreads();
    const int lane = threadIdx.x % WAVE, half = lane / 32;
    const int64_t step = (int64_t)gridDim.x * TRAIN_FW * TRAIN_ROWS;
    for (int64_t r0 = ((int64_t)blockIdx.x * TRAIN_FW + threadIdx.x / WAVE) * TRAIN_ROWS; r0 < rows; r0 += step) {
        const int64_t r = r0 + lane % 32;
        float f[MLP_IN];
#pragma unroll
        for (int q = 0; q < MLP_IN; ++q) f[q] = r < rows ? F[12 * r + q] : 0.f;
        uint4 h1[8];
        train_layer1(f, w1s, half, h1);
        float part = 0.f;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float16_t z = train_layer2(h1, reinterpret_cast<const uint4 *>(w2s), b2s, t, lane);
#pragma unroll
            for (int v = 0; v < 16; ++v)
                part = fmaf(w3s[unit(t, v, half)], bf16r(gelu_value(z[v], gelu_sigmoid(z[v]))), part);
        }
        part += __shfl_xor(part, 32, WAVE);
        if (half == 0 && r < rows) y[r] = part + P[P_B3];
    }
}

// per group (slice): q = softmax(y), loss += KL(p* || q), dy = q - p*
__global__ __launch_bounds__(256) void k_softmax_kl(const float *__restrict__ y, const float *__restrict__ pstar,
                                                    const int32_t *__restrict__ goff, float *__restrict__ dy,
                                                    float *__restrict__ loss) {
    __shared__ float red[256];
    const int g = blockIdx.x, t = threadIdx.x;
    const int b = goff[g], e = goff[g + 1];
    float mxv = -INFINITY;
    for (int r = b + t; r < e; r += 256) mxv = fmaxf(mxv, y[r]);
    red[t] = mxv;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (t < w) red[t] = fmaxf(red[t], red[t + w]);
        __syncthreads();
    }
    const float ym = red[0];
    __syncthreads();
    float se = 0.f;
    for (int r = b + t; r < e; r += 256) se += expf(y[r] - ym);
    red[t] = se;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (t < w) red[t] += red[t + w];
        __syncthreads();
    }
    const float lse = ym + logf(red[0]);
    __syncthreads();
    float l = 0.f;
    for (int r = b + t; r < e; r += 256) {
        const float lq = y[r] - lse;
        const float p = pstar[r];
        if (p > 0.f) l += p * (logf(p) - lq);
        dy[r] = expf(lq) - p;
    }
    red[t] = l;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (t < w) red[t] += red[t + w];
        __syncthreads();
    }
    if (t == 0) atomicAdd(loss, red[0]);
}

// sum over the 32 lanes of a half of 16 values per lane: lane l ends with the
// sum of value l % 16 (in every 16-lane row of the half alike)
__device__ __forceinline__ float half_sums(float (&a)[16], int lane) {
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) {
        const bool up = (lane & o) != 0;
#pragma unroll
        for (int k = 0; k < o; ++k) {
            const float give = up ? a[k] : a[k + o], keep = up ? a[k + o] : a[k];
            a[k] = keep + __shfl_xor(give, o, WAVE);
        }
    }
    return a[0] + __shfl_xor(a[0], 16, WAVE);
}

// Gradients of sum(dy * y) except dW2 and db2, straight-through at the bf16
// rounding points; dz2 (FP32) and h1 (bfloat16) of every row to the scratch.
__global__ __launch_bounds__(64 * TRAIN_BW) void k_train_backward(const float *__restrict__ P, int64_t rows,
                                                                  const float *__restrict__ F,
                                                                  const float *__restrict__ dy, float *__restrict__ dz2_out,
                                                                  uint16_t *__restrict__ h1_out, float *__restrict__ G) {
    constexpr int NT = 64 * TRAIN_BW;
    __shared__ __align__(16) uint16_t w2s[MLP_HID * MLP_HID], w2b[MLP_HID * MLP_HID];
    __shared__ __align__(16) float w1s[MLP_HID * TRAIN_W1];
    __shared__ float b2s[MLP_HID], w3s[MLP_HID];
    __shared__ __align__(16) float turn[TRAIN_BW][TRAIN_ROWS * TRAIN_LD];
    stage_w2<true>(P, w2s, NT);
    stage_w2<false>(P, w2b, NT);
    stage_w1(P, w1s, NT);
    for (int e = threadIdx.x; e < MLP_HID; e += NT) {
        b2s[e] = P[P_B2 + e];
        w3s[e] = bf16r(P[P_W3 + e]);
    }
    __syncthreads();
    const int lane = threadIdx.x % WAVE, half = lane / 32;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const uint4 *wf = reinterpret_cast<const uint4 *>(w2s), *wb = reinterpret_cast<const uint4 *>(w2b);
    float *tile = turn[w];
    f4_t g1[8];                       // dW1 and db1: units 16 i + 4 (lane / 16) + v, feature lane % 16 (12: the bias)
#pragma unroll
    for (int i = 0; i < 8; ++i) g1[i] = f4_t{0.f, 0.f, 0.f, 0.f};
    float gw3[4] = {0.f, 0.f, 0.f, 0.f}, gb3 = 0.f;
    const int64_t step = (int64_t)gridDim.x * TRAIN_BW * TRAIN_ROWS;
    for (int64_t r0 = ((int64_t)blockIdx.x * TRAIN_BW + w) * TRAIN_ROWS; r0 < rows; r0 += step) {
        const int64_t r = r0 + lane % 32;
        const bool in = r < rows;
        float f[MLP_IN];
#pragma unroll
        for (int q = 0; q < MLP_IN; ++q) f[q] = in ? F[12 * r + q] : 0.f;
        const float d = in ? dy[r] : 0.f;
        gb3 += d;
        uint4 h1[8];
        train_layer1(f, w1s, half, h1);
        if (in) {
#pragma unroll
            for (int st = 0; st < 8; ++st) {     // step st: units 32 (st / 2) + 16 (st % 2) + {0..3, 8..11} + 4 half
                uint16_t *o = h1_out + r * MLP_HID + unit(st / 2, 8 * (st % 2), half);
                *reinterpret_cast<uint2 *>(o) = make_uint2(h1[st].x, h1[st].y);
                *reinterpret_cast<uint2 *>(o + 8) = make_uint2(h1[st].z, h1[st].w);
            }
        }
        float16_t dh[4];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) dh[t][v] = 0.f;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float16_t z = train_layer2(h1, wf, b2s, t, lane);
            float dz[16], a3[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const GeluSigmoid sg = gelu_sigmoid(z[v]);
                a3[v] = d * bf16r(gelu_value(z[v], sg));
                dz[v] = d * w3s[unit(t, v, half)] * gelu_slope(z[v], sg);
            }
            if (r0 + TRAIN_ROWS > rows) {          // rows past the end add nothing, whatever the biases give there
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    a3[v] = in ? a3[v] : 0.f;
                    dz[v] = in ? dz[v] : 0.f;
                }
            }
            gw3[t] += half_sums(a3, lane);
            if (in) {
#pragma unroll
                for (int v = 0; v < 16; v += 4)
                    *reinterpret_cast<float4 *>(dz2_out + r * MLP_HID + unit(t, v, half)) =
                        make_float4(dz[v], dz[v + 1], dz[v + 2], dz[v + 3]);
            }
            // dh1 += W2^T dz2 over the tile's units, dz2 as three bfloat16 terms
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                uint4 term[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    uint32_t pk[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        float &x0 = dz[8 * u + 2 * k], &x1 = dz[8 * u + 2 * k + 1];
                        pk[k] = pack_bf16(x0, x1);
                        x0 = remainder_bf16(x0);
                        x1 = remainder_bf16(x1);
                    }
                    term[c] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
                }
#pragma unroll
                for (int tk = 0; tk < 4; ++tk) {
                    const uint4 a = wb[(tk * 8 + 2 * t + u) * 64 + lane];
                    dh[tk] = mfma_bf16(a, term[2], dh[tk]);
                    dh[tk] = mfma_bf16(a, term[1], dh[tk]);
                    dh[tk] = mfma_bf16(a, term[0], dh[tk]);
                }
            }
        }
        // dW1 and db1: dz1 of 32 units at a time through LDS, contracted over
        // the 32 rows with [features | 1] by v_mfma_f32_16x16x4
        float fb[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int64_t rr = r0 + 4 * k + lane / 16;
            const int q = lane % 16;
            fb[k] = rr < rows ? (q < MLP_IN ? F[12 * rr + q] : (q == MLP_IN ? 1.f : 0.f)) : 0.f;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
#pragma unroll
            for (int v = 0; v < 16; v += 4) {
                float dz[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {      // gelu' formed again: keeping it took 64 registers
                    const float z = train_z1(f, w1s, t, v + c, half);
                    dz[c] = dh[t][v + c] * gelu_slope(z, gelu_sigmoid(z));
                }
                *reinterpret_cast<float4 *>(tile + (lane % 32) * TRAIN_LD + unit(0, v, half)) =
                    make_float4(dz[0], dz[1], dz[2], dz[3]);
                __builtin_amdgcn_sched_barrier(0);
            }
            wave_lds_sync();
#pragma unroll
            for (int k = 0; k < 8; ++k)
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
                    g1[2 * t + mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                        tile[(4 * k + lane / 16) * TRAIN_LD + 16 * mt + lane % 16], fb[k], g1[2 * t + mt], 0, 0, 0);
            wave_lds_sync();
        }
    }
    // the workgroup's sums, wavefront by wavefront through LDS (w1s is done with), then one atomic per parameter
    __syncthreads();
    for (int e = threadIdx.x; e < MLP_HID * TRAIN_W1; e += NT) w1s[e] = 0.f;
    for (int e = threadIdx.x; e < MLP_HID; e += NT) w3s[e] = 0.f;
    __syncthreads();
    for (int ww = 0; ww < TRAIN_BW; ++ww) {
        if (ww == w) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) w1s[(16 * i + 4 * (lane / 16) + v) * TRAIN_W1 + lane % 16] += g1[i][v];
            if (lane % 32 < 16) {
#pragma unroll
                for (int t = 0; t < 4; ++t) w3s[unit(t, lane % 16, half)] += gw3[t];
            }
        }
        __syncthreads();
    }
    for (int e = threadIdx.x; e < MLP_HID * TRAIN_W1; e += NT) {
        const int k = e / TRAIN_W1, q = e % TRAIN_W1;
        if (q < MLP_IN) atomicAdd(G + P_W1 + k * MLP_IN + q, w1s[e]);
        if (q == MLP_IN) atomicAdd(G + P_B1 + k, w1s[e]);
    }
    for (int e = threadIdx.x; e < MLP_HID; e += NT) atomicAdd(G + P_W3 + e, w3s[e]);
    gb3 = half == 0 ? gb3 : 0.f;
#pragma unroll
    for (int o = 16; o >= 1; o >>= 1) gb3 += __shfl_xor(gb3, o, WAVE);
    if (lane == 0) atomicAdd(G + P_B3, gb3);
}

// dW2[h][k] = sum_r dz2[r][h] h1[r][k] and db2[h] = sum_r dz2[r][h] by
// v_mfma_f32_32x32x2: a wavefront owns 32 of the h and every k over the
// workgroup's rows, operands straight from the scratch (each load a whole
// 128- or 64-byte piece of a row), the next block of rows in flight.
constexpr int DW2_ROWS = 16;               // rows of a block
__global__ __launch_bounds__(256) void k_train_dw2(int64_t rows, int64_t per, const float *__restrict__ dz2,
                                                   const uint16_t *__restrict__ h1, float *__restrict__ G) {
    const int lane = threadIdx.x % WAVE, c = lane % 32, half = lane / 32;
    const int w = threadIdx.x / WAVE;
    const int64_t beg = blockIdx.x * per, end = min(rows, beg + per);
    float16_t acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
    float sum = 0.f;
    constexpr int NS = DW2_ROWS / 2;
    float an[NS];
    uint16_t bn[NS][4];
    auto load = [&](int64_t r0) {
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const int64_t r = r0 + 2 * i + half;
            const int64_t rc = r < end ? r : end - 1;
            an[i] = dz2[rc * MLP_HID + 32 * w + c];
#pragma unroll
            for (int t = 0; t < 4; ++t) bn[i][t] = h1[rc * MLP_HID + 32 * t + c];
        }
    };
    if (beg < end) load(beg);
    for (int64_t r0 = beg; r0 < end; r0 += DW2_ROWS) {
        float a[NS], b[NS][4];
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const bool in = r0 + 2 * i + half < end;
            a[i] = in ? an[i] : 0.f;
#pragma unroll
            for (int t = 0; t < 4; ++t) b[i][t] = in ? __uint_as_float((uint32_t)bn[i][t] << 16) : 0.f;
        }
        if (r0 + DW2_ROWS < end) load(r0 + DW2_ROWS);
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            sum += a[i];
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[i][t], acc[t], 0, 0, 0);
        }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            atomicAdd(G + P_W2 + (32 * w + unit(0, v, half)) * MLP_HID + 32 * t + c, acc[t][v]);
    sum += __shfl_xor(sum, 32, WAVE);
    if (half == 0) atomicAdd(G + P_B2 + 32 * w + c, sum);
}

// Adam (Kingma & Ba) with bias correction; step counts from 1
__global__ void k_adam(float *__restrict__ P, const float *__restrict__ G, float *__restrict__ M,
                       float *__restrict__ V, int32_t step, float lr) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= MLP_PARAMS) return;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float g = G[e];
    const float m = b1 * M[e] + (1.f - b1) * g;
    const float v = b2 * V[e] + (1.f - b2) * g * g;
    M[e] = m;
    V[e] = v;
    const float mh = m / (1.f - powf(b1, (float)step));
    const float vh = v / (1.f - powf(b2, (float)step));
    P[e] -= lr * mh / (sqrtf(vh) + eps);
}

__global__ void k_zero(float *p, int n) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) p[e] = 0.f;
}

unsigned blocks_for(int64_t n, int threads) { return (unsigned)((n + threads - 1) / threads); }

}  // namespace

int launch_features(hipStream_t st, const vplmc_plan &plan, const SliceDesc *desc, const vplmc_points &pts,
                    const int32_t *pt_ids, const int32_t *cl_ids, const float *lights, const float *bbox,
                    const vplmc_cut &cut, const int32_t *node_members, const int32_t *cnt, const float *mn,
                    const float *mx, const double *sum, const double *sumsq, const int32_t *zeros, float *slice_geo,
                    float *features) {
    if (plan.n_slices <= 0) return VPLMC_OK;
    hipLaunchKernelGGL(k_features, dim3(plan.n_slices), dim3(256), 0, st, desc, pts, pt_ids, cl_ids, lights,
                       plan.n_lights, bbox, cut, node_members, cnt, mn, mx, sum, sumsq, zeros, slice_geo, features);
    VPLMC_HIP(hipGetLastError());
    return VPLMC_OK;
}

int launch_mlp_forward(hipStream_t st, const float *params, int64_t rows, const float *features, float *y) {
    if (rows <= 0) return VPLMC_OK;
    hipLaunchKernelGGL(k_mlp_forward, dim3(blocks_for(rows, 128)), dim3(256), 0, st, params, rows, features, y);
    VPLMC_HIP(hipGetLastError());
    return VPLMC_OK;
}

// workgroups of a training pass: a wavefront per 32 rows, at most MAX_TRAIN_GRID
// (they walk the rows, so that weights are staged and gradients added once per workgroup)
constexpr int64_t MAX_TRAIN_GRID = 256;

static int launch_train_backward(hipStream_t st, const float *params, int64_t rows, const float *features,
                                 const float *dy, float *grad, float *cache) {
    // the scratch is aligned for floats only; its activation part holds 512 floats per row, of which dz2
    // and h1 take 192
    float *dz2 = reinterpret_cast<float *>((reinterpret_cast<uintptr_t>(cache) + 15) & ~(uintptr_t)15);
    uint16_t *h1 = reinterpret_cast<uint16_t *>(dz2 + rows * MLP_HID);
    const int64_t grid = std::min<int64_t>((rows + TRAIN_BW * TRAIN_ROWS - 1) / (TRAIN_BW * TRAIN_ROWS), MAX_TRAIN_GRID);
    hipLaunchKernelGGL(k_train_backward, dim3((unsigned)grid), dim3(64 * TRAIN_BW), 0, st, params, rows, features, dy,
                       dz2, h1, grad);
    VPLMC_HIP(hipGetLastError());
    // one workgroup per CU: twice as many took 79 us instead of 75 at 131,072 rows (each adds 16,512 sums)
    const int64_t per = std::max<int64_t>((rows + MAX_TRAIN_GRID - 1) / MAX_TRAIN_GRID, 4 * DW2_ROWS);
    hipLaunchKernelGGL(k_train_dw2, dim3((unsigned)((rows + per - 1) / per)), dim3(256), 0, st, rows, per, dz2, h1, grad);
    VPLMC_HIP(hipGetLastError());
    return VPLMC_OK;
}

int launch_mlp_grad(hipStream_t st, const float *params, int64_t rows, const float *features, const float *dy,
                    float *grad, float *cache) {
    hipLaunchKernelGGL(k_zero, dim3(blocks_for(MLP_PARAMS, 256)), dim3(256), 0, st, grad, MLP_PARAMS);
    VPLMC_HIP(hipGetLastError());
    if (rows <= 0) return VPLMC_OK;
    return launch_train_backward(st, params, rows, features, dy, grad, cache);
}

int launch_mlp_train_step(hipStream_t st, float *params, float *m, float *v, int32_t step, float lr, int64_t rows,
                          const float *features, const float *pstar, int32_t n_groups, const int32_t *group_off,
                          float *y, float *dy, float *grad, float *loss, float *cache) {
    hipLaunchKernelGGL(k_zero, dim3(blocks_for(MLP_PARAMS, 256)), dim3(256), 0, st, grad, MLP_PARAMS);
    hipLaunchKernelGGL(k_zero, dim3(1), dim3(32), 0, st, loss, 1);
    VPLMC_HIP(hipGetLastError());
    if (rows > 0) {
        const int64_t grid =
            std::min<int64_t>((rows + TRAIN_FW * TRAIN_ROWS - 1) / (TRAIN_FW * TRAIN_ROWS), 3 * MAX_TRAIN_GRID);
        hipLaunchKernelGGL(k_train_forward, dim3((unsigned)grid), dim3(64 * TRAIN_FW), 0, st, params, rows, features, y);
        hipLaunchKernelGGL(k_softmax_kl, dim3(n_groups), dim3(256), 0, st, y, pstar, group_off, dy, loss);
        VPLMC_HIP(hipGetLastError());
        int rc = launch_train_backward(st, params, rows, features, dy, grad, cache);
        if (rc) return rc;
    }
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(MLP_PARAMS, 256)), dim3(256), 0, st, params, grad, m, v, step, lr);
    VPLMC_HIP(hipGetLastError());
    return VPLMC_OK;
}

int launch_mlp_adam(hipStream_t st, float *params, const float *grad, float *m, float *v, int32_t step, float lr) {
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(MLP_PARAMS, 256)), dim3(256), 0, st, params, grad, m, v, step, lr);
    VPLMC_HIP(hipGetLastError());
    return VPLMC_OK;
}

}  // namespace vplmc
