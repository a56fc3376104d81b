// Per-row masked alternating least squares: a completion variant of the
// slice matrix beside the ADM (Appendix A).  Every row of X, then every
// column of Y, is the ridge least-squares fit to its own observed entries
// (weighted regularisation, Zhou et al. 2008):
//
//   x_i = (sum_{c in Omega_i} y_c y_c^T + lam max(1, n_i) I)^-1 sum_{c in Omega_i} M_ic y_c
//   y_c = (sum_{i in Omega^c} x_i x_i^T + lam max(1, n_c) I)^-1 sum_{i in Omega^c} M_ic x_i
//
// on the stacked m' x 3n' matrix (a sample (i, j) observes columns j, n + j
// and 2n + j, so n_i is three times the row's samples and the three channel
// columns of j share one Gram matrix).  Same scale s0, initial factors,
// residual test and iteration cap as the ADM; components past the slice's
// rank stay 0 (their Gram block is lam max(1, n) I and their right-hand side
// 0).
//
// Two launches per iteration over all slices of a rank bucket (k_als_rows,
// k_als_cols), after an init launch and before a final one, so that a frame of
// a few dozen slices fills the chip and the launch boundaries order the
// half-steps (with the residual stop also a loop over the iterations, see
// ALS_LAUNCHED).  A 16-lane row of a wavefront (32 lanes at rank 32) owns one
// system, lane r holding row r of its Gram: a factor vector is one coalesced
// load of the tile, and each lane multiplies its own component by every
// component, broadcast by DPP.  The Gram is summed in FP32 in sample order;
// each lane then turns its row to FP64 and the tile solves by Gauss-Jordan
// elimination (symmetric positive definite, so no pivoting), the pivot row
// broadcast by DPP as well, so the system never leaves the registers.  The
// loads run two blocks of samples ahead of the arithmetic (index, then the
// vectors it names).  The init launch orders a slice's rows and columns by
// decreasing sample count: the systems of a wavefront are then of similar
// length, and the longest start first.
// The residual of the iterate that enters an iteration is formed by the row
// launch from the Y vectors it loads anyway; its sums per workgroup land in
// slots, which every workgroup of the column launch adds in slot order for
// the stop test.  The row launch writes the second X buffer, so a slice that
// stops keeps the X its residual was measured on.  Every system is summed in
// sample order, and a row's place in a slot's sum depends on the counts alone:
// factors, residuals and iteration counts are bit-reproducible.
//
// The row launch is bound by VALU issue (0.62 busy: Grams, elimination), the
// column launch by the gathers and the dependent chain of its longest sums (0.21
// busy, 0.7 wavefronts per SIMD).  Measured on one MI355X, 48 slices of
// 200-900 rows, 300 columns, rank 16, 6.5% sampled, 100 iterations: 467 ms
// with one 512-thread workgroup per slice and the systems in LDS (Cholesky by
// one wavefront per row), 11.8 ms now; Grams on the matrix unit (a
// wavefront per four systems, summed in another order) took 16 ms in FP32 and
// 26 ms in FP64.

#include <algorithm>
#include <utility>

#include "vplmc_internal.h"

namespace vplmc {
namespace {

constexpr int WAVE = 64;
constexpr int ALS_THREADS = 256;      // of the row and column launches
constexpr int ALS_NW = ALS_THREADS / WAVE;
constexpr int ALS_LOOP_THREADS = 512;
// With the residual stop, the launches after the last slice has stopped still
// cost 2.7 us each.  So at most ALS_LAUNCHED iterations are launches, and one
// launch of k_als_loop, a workgroup per slice, does what is left (limit 2,000,
// stopped after one: 15.0 -> 0.7 ms); the default limit of 100 lies below.
// Slices so small that a workgroup per slice does well are its from the start:
// up to ALS_LOOP_EDGE rows and columns (64 x 32, rank 8: 178 us against 680
// stopped after two iterations, 2.0 ms against 1.6 after 100; 16 of 64 x 64, rank
// 16: 0.27 / 0.69 and 5.2 / 2.8 ms), twice that where ALS_LOOP_MANY slices fill
// the chip (400 of 128 x 128, rank 16: 0.54 / 1.57 and 14.9 / 15.9 ms).  Rank 32
// (64 x 64: 0.56 / 0.72, 27 / 6 ms) and fixed counts stay with the launches.
constexpr int ALS_LAUNCHED = 128;
constexpr int ALS_LOOP_EDGE = 64, ALS_LOOP_MANY = 400;
constexpr int ALS_INIT_THREADS = 512;
constexpr int ALS_BINS = 1024;        // sample counts told apart by the ordering

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, WAVE);
    return v;
}

// sum over the block of one double per thread, in a fixed order
template <int NW>
__device__ __forceinline__ double block_sum_d(double v, double *red) {
    const int t = threadIdx.x, lane = t % WAVE, w = t / WAVE;
    v = wave_sum_d(v);
    if (lane == 0) red[w] = v;
    __syncthreads();
    double s = 0.0;
    for (int k = 0; k < NW; ++k) s += red[k];
    __syncthreads();
    return s;
}

// how a rank is laid out on a wavefront
template <int Q>
struct AlsShape {
    static constexpr int T = Q <= 16 ? 16 : 32;         // lanes of a system
    static constexpr int SYS = WAVE / T;                // systems per wavefront
    static constexpr int GRP = SYS * ALS_NW;            // systems per workgroup
    // workgroups per row block of the plan (per column block: its columns / GRP)
    static constexpr int RSUB = GADM_RB / GRP;
};

// per-slice state between the launches
struct AlsState {
    int32_t done, iters, resid, zero;    // resid: FP32 bits; zero: every sample is 0
    double norm_m, s0;                   // ||P_Omega M|| / s0, mean sampled value
};

struct AlsArgs {
    const SliceDesc *desc;
    const int32_t *ids;                  // the group's slices
    const int32_t *rowp, *colp;          // count + 1: prefixes of the slices' row and column blocks
    int32_t count;
    uint64_t seed;
    int32_t max_iter, mode;
    float tol, lam;
    const int32_t *row_ptr_all, *csr_col_all;
    const float *csr_val_all;
    const int32_t *col_ptr_all, *csc_row_all;
    const float *csc_val_all;
    float *X_all, *Xn_all, *Y_all, *scale_all;
    int32_t *rord_all, *cord_all;        // per slice at off_x, off_y: its rows and columns by decreasing count
    int32_t *stats_all;
    char *gsys;
    double *e2;                          // RSUB slots per row block of the group
    int32_t cb;                          // columns per column block
};

__device__ __forceinline__ AlsState *state_of(char *base, int s) {
    return reinterpret_cast<AlsState *>(base + (size_t)s * GADM_SYS_BYTES);
}

// the slice position k with pre[k] <= b < pre[k + 1]
__device__ __forceinline__ int block_slice(const int32_t *__restrict__ pre, int count, int b) {
    int lo = 0, hi = count;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (pre[mid] <= b) lo = mid; else hi = mid;
    }
    return lo;
}

// the items 0 .. n - 1 of a CSR / CSC pointer by decreasing count (counts past
// ALS_BINS - 1 alike), equal counts in index order: a system's workgroup, and
// with it the order of the residual's sum, is the same in every run.  A chunk
// of items at a time, each counting the equal ones before it.  All threads call.
struct AlsOrder {
    int32_t bins[ALS_BINS];
    __align__(16) uint16_t chunk[ALS_INIT_THREADS];
};
__device__ void order_by_count(const int32_t *__restrict__ ptr, int n, int32_t *__restrict__ order, AlsOrder &sh) {
    const int t = threadIdx.x;
    int32_t *bins = sh.bins;
    auto bin = [&](int i) { return ALS_BINS - 1 - min(ptr[i + 1] - ptr[i], ALS_BINS - 1); };
    for (int e = t; e < ALS_BINS; e += ALS_INIT_THREADS) bins[e] = 0;
    __syncthreads();
    for (int i = t; i < n; i += ALS_INIT_THREADS) atomicAdd(bins + bin(i), 1);
    __syncthreads();
    if (t < WAVE) {                       // exclusive prefix on one wavefront
        constexpr int PER = ALS_BINS / WAVE;
        int sum = 0;
        for (int e = 0; e < PER; ++e) sum += bins[t * PER + e];
        int incl = sum;
        for (int o = 1; o < WAVE; o <<= 1) {
            const int u = __shfl_up(incl, o, WAVE);
            if (t >= o) incl += u;
        }
        int base = incl - sum;
        for (int e = 0; e < PER; ++e) {
            const int c = bins[t * PER + e];
            bins[t * PER + e] = base;
            base += c;
        }
    }
    for (int i0 = 0; i0 < n; i0 += ALS_INIT_THREADS) {
        const int i = i0 + t;
        const int b = i < n ? bin(i) : 0xFFFF;
        sh.chunk[t] = (uint16_t)b;
        __syncthreads();
        int before = 0, equal = 0;
#pragma unroll 4
        for (int u = 0; u < ALS_INIT_THREADS; u += 8) {
            const uint4 v = *reinterpret_cast<const uint4 *>(sh.chunk + u);
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int same = (int)((w[k / 2] >> (k % 2 * 16)) & 0xFFFFu) == b ? 1 : 0;
                equal += same;
                before += u + k < t ? same : 0;
            }
        }
        const int at = i < n ? bins[b] + before : 0;
        __syncthreads();
        if (i < n) {
            order[at] = i;
            if (before + 1 == equal) bins[b] = at + 1;     // the last of its count in the chunk
        }
        __syncthreads();
    }
}

// scale s0 = mean sampled value, ||P_Omega M|| of M / s0, initial factors as the ADM's
template <int Q>
__global__ __launch_bounds__(ALS_INIT_THREADS) void k_als_init(AlsArgs a) {
    __shared__ double red[ALS_INIT_THREADS / WAVE];
    __shared__ AlsOrder ord;
    const int s = __builtin_amdgcn_readfirstlane(a.ids[blockIdx.x]);
    const SliceDesc d = a.desc[s];
    const int m = d.m, n = d.n, qr = d.qr, t = threadIdx.x;
    const float *csr_val = a.csr_val_all + 3 * d.off_omega;
    float *X = a.X_all + d.off_x;
    float *Y = a.Y_all + d.off_y;
    AlsState *st = state_of(a.gsys, s);
    const int nnz = a.row_ptr_all[d.off_row + m];
    double sum = 0.0, sumsq = 0.0;
    for (int p = t; p < 3 * nnz; p += ALS_INIT_THREADS) {
        const double v = (double)csr_val[p];
        sum += v;
        sumsq += v * v;
    }
    sum = block_sum_d<ALS_INIT_THREADS / WAVE>(sum, red);
    sumsq = block_sum_d<ALS_INIT_THREADS / WAVE>(sumsq, red);
    const bool zero = nnz == 0 || !(sumsq > 0.0);
    const double s0 = zero ? 0.0 : sum / (3.0 * (double)nnz);
    if (t == 0) {
        st->done = zero ? 1 : 0;
        st->iters = zero ? 0 : a.max_iter;
        st->resid = 0;
        st->zero = zero ? 1 : 0;
        st->norm_m = zero ? 0.0 : sqrt(sumsq) / s0;
        st->s0 = s0;
        a.scale_all[s] = (float)s0;
    }
    order_by_count(a.row_ptr_all + d.off_row, m, a.rord_all + d.off_x, ord);
    order_by_count(a.col_ptr_all + d.off_colptr, n, a.cord_all + d.off_y, ord);
    const float cq = (float)(2.0 / sqrt((double)qr));
    const bool given = (a.mode & 2) != 0;
    for (int e = t; e < m * Q; e += ALS_INIT_THREADS) {
        const int i = e / Q, k = e % Q;
        float v = 0.f;
        if (!zero && k < qr)
            v = given ? X[e]
                      : __fmul_rn((float)(philox(a.seed, (uint64_t)s, (uint64_t)i, (uint64_t)k, TAG_INITX, 0).a >> 40) *
                                      0x1p-24f,
                                  cq);
        X[e] = v;
    }
    for (int e = t; e < 3 * n * Q; e += ALS_INIT_THREADS) {
        const int j = e / (3 * Q), c = (e / Q) % 3, k = e % Q;
        float v = 0.f;
        if (!zero && k < qr) {
            const uint64_t col = (uint64_t)c * (uint64_t)n + (uint64_t)j;
            v = given ? Y[e]
                      : __fmul_rn((float)(philox(a.seed, (uint64_t)s, (uint64_t)k, col, TAG_INITY, 0).a >> 40) *
                                      0x1p-24f,
                                  cq);
        }
        Y[e] = v;
    }
}

// sum over the lanes of each tile, the same bits in all of them
template <int T>
__device__ __forceinline__ float tile_sum(float v) {
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));   // quad_perm [1 0 3 2]
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true));   // quad_perm [2 3 0 1]
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, true));  // row_half_mirror
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xF, 0xF, true));  // row_mirror
    if constexpr (T == 32) v += __shfl_xor(v, 16, WAVE);
    return v;
}

// lane J's value of each 16-lane row (T = 16: DPP row_newbcast) or 32-lane half
template <int T, int J>
__device__ __forceinline__ double tile_bcast(double v) {
    if constexpr (T == 16) {
        const long long b = __double_as_longlong(v);
        const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x150 + J, 0xF, 0xF, true);
        const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x150 + J, 0xF, 0xF, true);
        return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
    } else {
        return __shfl(v, J, 32);
    }
}

template <int J>
__device__ __forceinline__ float row_bcast(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + J, 0xF, 0xF, true));
}

template <int J>
__device__ __forceinline__ int row_bcast(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0x150 + J, 0xF, 0xF, true);
}
// f(0), ..., f(U - 1) with constant arguments (a DPP lane number is one)
template <int U, typename F, int... I>
__device__ __forceinline__ void block_u_(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int U, typename F>
__device__ __forceinline__ void block_u(F &&f) {
    block_u_<U>(f, std::make_integer_sequence<int, U>{});
}

// one component of a vector per lane of a tile -> its 16-component blocks,
// each held alike by every 16-lane row of the tile
template <int T>
__device__ __forceinline__ void blocks_of(float v, int r, float (&blk)[T / 16]) {
    if constexpr (T == 16) {
        blk[0] = v;
    } else {
        const float o = __shfl_xor(v, 16, WAVE);
        blk[0] = r < 16 ? v : o;
        blk[1] = r < 16 ? o : v;
    }
}

// G[k] += f f_k (columns), or with the three channels of a sample
// G[k] += (f1 f1_k + f0 f0_k) + f2 f2_k, rounded in that order
template <int Q, int T, int K>
__device__ __forceinline__ void gram_add(float (&G)[Q], float f, const float (&b)[T / 16]) {
    if constexpr (K < Q) {
        G[K] = fmaf(f, row_bcast<K % 16>(b[K / 16]), G[K]);
        gram_add<Q, T, K + 1>(G, f, b);
    }
}
template <int Q, int T, int K>
__device__ __forceinline__ void gram_add3(float (&G)[Q], const float (&f)[3], const float (&b)[3][T / 16]) {
    if constexpr (K < Q) {
        const float p = fmaf(f[0], row_bcast<K % 16>(b[0][K / 16]), __fmul_rn(f[1], row_bcast<K % 16>(b[1][K / 16])));
        G[K] = __fadd_rn(G[K], fmaf(f[2], row_bcast<K % 16>(b[2][K / 16]), p));
        gram_add3<Q, T, K + 1>(G, f, b);
    }
}

// step J of the elimination: row J is the pivot row, every other row of the
// tile loses its component J (components below J are not needed any more)
template <int Q, int T, int NR, int J>
__device__ __forceinline__ void gj_steps(double (&A)[Q], double (&b)[NR], double &dinv, int r) {
    if constexpr (J < Q) {
        const double inv = 1.0 / tile_bcast<T, J>(A[J]);
        const double f = r == J ? 0.0 : A[J] * inv;
        dinv = r == J ? inv : dinv;
#pragma unroll
        for (int k = J + 1; k < Q; ++k) A[k] = fma(-f, tile_bcast<T, J>(A[k]), A[k]);
#pragma unroll
        for (int c = 0; c < NR; ++c) b[c] = fma(-f, tile_bcast<T, J>(b[c]), b[c]);
        gj_steps<Q, T, NR, J + 1>(A, b, dinv, r);
    }
}

// (G + shift I)^-1 b of the systems of a wavefront, lane r of a tile holding
// row r of its system's G and component r of the right-hand sides
template <int Q, int NR>
__device__ __forceinline__ void tile_solve(const float (&G)[Q], double shift, double (&b)[NR], int r) {
    using S = AlsShape<Q>;
    double A[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) A[k] = (double)G[k];
#pragma unroll
    for (int k = 0; k < Q; ++k) A[k] += r == k ? shift : 0.0;
    double dinv = 0.0;
    gj_steps<Q, S::T, NR, 0>(A, b, dinv, r);
#pragma unroll
    for (int c = 0; c < NR; ++c) b[c] *= dinv;
}

// One row per tile of the wavefront: the row at place `at` of the slice's order
// (none past the last).  Lane 0 of the tile returns its squared residual of the
// iterate that enters iteration it.
template <int Q>
__device__ __forceinline__ double als_row(const AlsArgs &a, const SliceDesc &d, float inv_s0, int it, int at) {
    using S = AlsShape<Q>;
    constexpr int U = 8;                             // samples of a block
    const int lane = threadIdx.x % WAVE, r = lane % S::T;
    const int32_t *row_ptr = a.row_ptr_all + d.off_row;
    const int32_t *csr_col = a.csr_col_all + d.off_omega;
    const float *csr_val = a.csr_val_all + 3 * d.off_omega;
    const float *X = ((it & 1) ? a.Xn_all : a.X_all) + d.off_x;
    float *Xn = ((it & 1) ? a.X_all : a.Xn_all) + d.off_x;
    const float *Y = a.Y_all + d.off_y;
    const bool in = at < d.m, comp = r < Q;
    const int i = in ? a.rord_all[d.off_x + at] : 0;
    const int p0 = in ? row_ptr[i] : 0, cnt = in ? row_ptr[i + 1] - p0 : 0;
    int most = cnt;                                  // longest of the wavefront's systems
#pragma unroll
    for (int o = S::T; o < WAVE; o <<= 1) most = max(most, __shfl_xor(most, o, WAVE));
    most = __builtin_amdgcn_readfirstlane(most);
    const float x = in && comp ? X[(size_t)i * Q + r] : 0.f;
    float G[Q], rhs = 0.f;
#pragma unroll
    for (int k = 0; k < Q; ++k) G[k] = 0.f;
    double e2 = 0.0;
    // lane l of a 16-lane row holds the index and the values of sample l % U
    // of a block; past the end a lane reads the slice's first sample (every
    // slice in this launch has one) and its vectors are taken as 0
    int jn;
    float y[U][3], vn[3], vc[3];
    const int su = lane % U;
    auto load_index = [&](int e0) {
        const int p = e0 + su < cnt ? p0 + e0 + su : 0;
        jn = csr_col[p];
#pragma unroll
        for (int c = 0; c < 3; ++c) vn[c] = csr_val[3 * (size_t)p + c];
    };
    auto load_block = [&]() {                        // the samples whose indices are in jn
        block_u<U>([&](auto u) {
            const float *yj = Y + (size_t)row_bcast<u.value>(jn) * 3 * Q + (comp ? r : 0);
#pragma unroll
            for (int c = 0; c < 3; ++c) y[u.value][c] = yj[c * Q];
        });
    };
    load_index(0);
    load_block();
    for (int e0 = 0; e0 < most; e0 += U) {
        float yb[U][3];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < 3; ++c) yb[u][c] = e0 + u < cnt && comp ? y[u][c] : 0.f;
#pragma unroll
        for (int c = 0; c < 3; ++c) vc[c] = e0 + su < cnt ? vn[c] * inv_s0 : 0.f;
        if (e0 + U < most) {
            load_index(e0 + U);
            load_block();
        }
        block_u<U>([&](auto uc) {
            constexpr int u = uc.value;
            float b[3][S::T / 16], mb[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                blocks_of<S::T>(yb[u][c], r, b[c]);
                mb[c] = row_bcast<u>(vc[c]);
            }
            gram_add3<Q, S::T, 0>(G, yb[u], b);
            rhs = __fadd_rn(rhs, fmaf(mb[2], yb[u][2], fmaf(mb[0], yb[u][0], __fmul_rn(mb[1], yb[u][1]))));
            const float xu = e0 + u < cnt ? x : 0.f;   // past the end the row's x may be anything
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float e = mb[c] - tile_sum<S::T>(xu * yb[u][c]);
                e2 = fma((double)e, (double)e, e2);
            }
        });
    }
    double b[1] = {(double)rhs};
    tile_solve<Q, 1>(G, in ? (double)a.lam * (double)max(1, 3 * cnt) : 1.0, b, r);
    if (in && comp) Xn[(size_t)i * Q + r] = r < d.qr ? (float)b[0] : 0.f;
    return r == 0 ? e2 : 0.0;
}

// Row half-step: GRP rows of one slice per workgroup.
template <int Q>
__global__ __launch_bounds__(ALS_THREADS) void k_als_rows(AlsArgs a, int it) {
    using S = AlsShape<Q>;
    __shared__ double red[ALS_NW];
    const int blk = blockIdx.x / S::RSUB, sub = blockIdx.x % S::RSUB;
    const int kk = block_slice(a.rowp, a.count, blk);
    const int s = __builtin_amdgcn_readfirstlane(a.ids[kk]);
    const AlsState *st = state_of(a.gsys, s);
    if (st->done) return;
    const SliceDesc d = a.desc[s];
    const int t = threadIdx.x, g = t % WAVE / S::T;
    const int w = __builtin_amdgcn_readfirstlane(t / WAVE);
    const int at = (blk - a.rowp[kk]) * GADM_RB + sub * S::GRP + w * S::SYS + g;   // the tile's place in the order
    const double e2 = block_sum_d<ALS_NW>(als_row<Q>(a, d, (float)(1.0 / st->s0), it, at), red);
    if (t == 0) a.e2[blockIdx.x] = e2;
}

// One column per tile: the column at place `at`, its three channels sharing a system.
template <int Q>
__device__ __forceinline__ void als_col(const AlsArgs &a, const SliceDesc &d, float inv_s0, int it, int at) {
    using S = AlsShape<Q>;
    constexpr int U = 16;                            // samples of a block
    const int lane = threadIdx.x % WAVE, r = lane % S::T;
    const int32_t *col_ptr = a.col_ptr_all + d.off_colptr;
    const int32_t *csc_row = a.csc_row_all + d.off_omega;
    const float *csc_val = a.csc_val_all + 3 * d.off_omega;
    const float *Xn = ((it & 1) ? a.X_all : a.Xn_all) + d.off_x;
    float *Y = a.Y_all + d.off_y;
    const bool in = at < d.n, comp = r < Q;
    const int j = in ? a.cord_all[d.off_y + at] : 0;
    const int p0 = in ? col_ptr[j] : 0, cnt = in ? col_ptr[j + 1] - p0 : 0;
    int most = cnt;
#pragma unroll
    for (int o = S::T; o < WAVE; o <<= 1) most = max(most, __shfl_xor(most, o, WAVE));
    most = __builtin_amdgcn_readfirstlane(most);
    float G[Q], rhs[3] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < Q; ++k) G[k] = 0.f;
    int jn;                                          // as in the row launch
    float x[U], vn[3], vc[3];
    const int su = lane % U;
    auto load_index = [&](int e0) {
        const int p = e0 + su < cnt ? p0 + e0 + su : 0;
        jn = csc_row[p];
#pragma unroll
        for (int c = 0; c < 3; ++c) vn[c] = csc_val[3 * (size_t)p + c];
    };
    auto load_block = [&]() {
        block_u<U>([&](auto u) { x[u.value] = Xn[(size_t)row_bcast<u.value>(jn) * Q + (comp ? r : 0)]; });
    };
    load_index(0);
    load_block();
    for (int e0 = 0; e0 < most; e0 += U) {
        float xb[U];
#pragma unroll
        for (int u = 0; u < U; ++u) xb[u] = e0 + u < cnt && comp ? x[u] : 0.f;
#pragma unroll
        for (int c = 0; c < 3; ++c) vc[c] = e0 + su < cnt ? vn[c] * inv_s0 : 0.f;
        if (e0 + U < most) {
            load_index(e0 + U);
            load_block();
        }
        block_u<U>([&](auto uc) {
            constexpr int u = uc.value;
            float b[S::T / 16];
            blocks_of<S::T>(xb[u], r, b);
            gram_add<Q, S::T, 0>(G, xb[u], b);
#pragma unroll
            for (int c = 0; c < 3; ++c) rhs[c] = fmaf(xb[u], row_bcast<u>(vc[c]), rhs[c]);
        });
    }
    double b[3] = {(double)rhs[0], (double)rhs[1], (double)rhs[2]};
    tile_solve<Q, 3>(G, in ? (double)a.lam * (double)max(1, cnt) : 1.0, b, r);
    if (in && comp) {
#pragma unroll
        for (int c = 0; c < 3; ++c) Y[(size_t)j * 3 * Q + c * Q + r] = r < d.qr ? (float)b[c] : 0.f;
    }
}

// Column half-step: GRP columns of one slice per workgroup; first the stop
// test on the residual slots.
template <int Q>
__global__ __launch_bounds__(ALS_THREADS) void k_als_cols(AlsArgs a, int it) {
    using S = AlsShape<Q>;
    __shared__ double red[ALS_NW];
    __shared__ int done_s;
    const int csub = a.cb / S::GRP, blk = blockIdx.x / csub, sub = blockIdx.x % csub;
    const int kk = block_slice(a.colp, a.count, blk);
    const int s = __builtin_amdgcn_readfirstlane(a.ids[kk]);
    AlsState *st = state_of(a.gsys, s);
    const SliceDesc d = a.desc[s];
    const int first_at = (blk - a.colp[kk]) * a.cb + sub * S::GRP;
    if (first_at >= d.n) return;
    // a slice that stops in this launch is marked by its first workgroup; the
    // others find the same sum, so it does not matter which they see first
    const int t = threadIdx.x, g = t % WAVE / S::T;
    if (t == 0) done_s = __hip_atomic_load(&st->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (done_s) return;
    if (!(a.mode & 1) || first_at == 0) {
        double e2 = 0.0;
        for (int u = a.rowp[kk] * S::RSUB + t; u < a.rowp[kk + 1] * S::RSUB; u += ALS_THREADS) e2 += a.e2[u];
        e2 = block_sum_d<ALS_NW>(e2, red);
        const double err = sqrt(e2) / st->norm_m;
        const bool stop = !(a.mode & 1) && err < (double)a.tol;
        if (first_at == 0 && t == 0) {
            st->resid = __float_as_int((float)err);
            if (stop) {
                st->iters = it;
                __hip_atomic_store(&st->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (stop) return;
    }
    const int w = __builtin_amdgcn_readfirstlane(t / WAVE);
    als_col<Q>(a, d, (float)(1.0 / st->s0), it, first_at + w * S::SYS + g);
}

// The iterations from it0 on, one workgroup per slice, until the slice stops.
template <int Q>
__global__ __launch_bounds__(ALS_LOOP_THREADS) void k_als_loop(AlsArgs a, int it0) {
    using S = AlsShape<Q>;
    constexpr int NW = ALS_LOOP_THREADS / WAVE;
    __shared__ double red[NW];
    const int s = __builtin_amdgcn_readfirstlane(a.ids[blockIdx.x]);
    AlsState *st = state_of(a.gsys, s);
    if (st->done) return;
    const SliceDesc d = a.desc[s];
    const int t = threadIdx.x, g = t % WAVE / S::T;
    const int w = __builtin_amdgcn_readfirstlane(t / WAVE);
    const float inv_s0 = (float)(1.0 / st->s0);
    const double norm_m = st->norm_m;
    for (int it = it0; it < a.max_iter; ++it) {
        double e2 = 0.0;
        for (int r0 = w * S::SYS; r0 < d.m; r0 += NW * S::SYS) e2 += als_row<Q>(a, d, inv_s0, it, r0 + g);
        e2 = block_sum_d<NW>(e2, red);
        const double err = sqrt(e2) / norm_m;
        const bool stop = !(a.mode & 1) && err < (double)a.tol;
        if (t == 0) {
            st->resid = __float_as_int((float)err);
            if (stop) st->iters = it;
        }
        if (stop) return;
        __threadfence_block();           // the new X before its columns read it
        __syncthreads();
        for (int c0 = w * S::SYS; c0 < d.n; c0 += NW * S::SYS) als_col<Q>(a, d, inv_s0, it, c0 + g);
        __threadfence_block();
        __syncthreads();
    }
}

// the final X into the X region, statistics
template <int Q>
__global__ __launch_bounds__(ALS_THREADS) void k_als_final(AlsArgs a) {
    const int s = __builtin_amdgcn_readfirstlane(a.ids[blockIdx.x]);
    const AlsState *st = state_of(a.gsys, s);
    const SliceDesc d = a.desc[s];
    const int t = threadIdx.x;
    if (st->iters & 1) {
        const float *src = a.Xn_all + d.off_x;
        float *dst = a.X_all + d.off_x;
        for (int e = t; e < d.m * Q; e += ALS_THREADS) dst[e] = src[e];
    }
    if (t == 0) {
        int32_t *o = a.stats_all + 4 * s;
        o[0] = st->iters;
        if (st->zero)
            o[1] |= VPLMC_SLICE_ALL_ZERO;
        else if (!(a.mode & 1) && st->iters >= a.max_iter)
            o[1] |= VPLMC_SLICE_NOT_CONVERGED;
        o[2] = st->resid;
    }
}

template <int Q>
int launch_als_q(hipStream_t st, const AlsArgs &args, const vplmc_plan &plan, int grp, const int32_t *gblk_dev,
                 double *e2) {
    using S = AlsShape<Q>;
    const size_t count = plan.groups[grp].size();
    if (count == 0) return VPLMC_OK;
    AlsArgs a = args;
    a.count = (int32_t)count;
    a.cb = plan.g_cb[grp];
    a.rowp = gblk_dev + plan.gblk_off[grp];
    a.colp = a.rowp + count + 1;
    a.e2 = e2 + ALS_E2_SLOTS * plan.ge2_base[grp];
    static_assert(S::RSUB <= ALS_E2_SLOTS, "residual slots of a row block");
    const unsigned nr = (unsigned)(plan.g_rows[grp] * S::RSUB), nc = (unsigned)(plan.g_cols[grp] * (a.cb / S::GRP));
    hipLaunchKernelGGL(k_als_init<Q>, dim3((unsigned)count), dim3(ALS_INIT_THREADS), 0, st, a);
    VPLMC_HIP(hipGetLastError());
    const int edge = (count >= (size_t)ALS_LOOP_MANY ? 2 : 1) * ALS_LOOP_EDGE;
    const bool small = Q <= 16 && plan.group_max_m[grp] <= edge && plan.group_max_n[grp] <= edge;
    const int launched = a.mode & 1 ? a.max_iter : small ? 0 : std::min(a.max_iter, ALS_LAUNCHED);
    for (int it = 0; it < launched; ++it) {
        hipLaunchKernelGGL(k_als_rows<Q>, dim3(nr), dim3(ALS_THREADS), 0, st, a, it);
        VPLMC_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_als_cols<Q>, dim3(nc), dim3(ALS_THREADS), 0, st, a, it);
        VPLMC_HIP(hipGetLastError());
    }
    if (launched < a.max_iter) {
        hipLaunchKernelGGL(k_als_loop<Q>, dim3((unsigned)count), dim3(ALS_LOOP_THREADS), 0, st, a, launched);
        VPLMC_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(k_als_final<Q>, dim3((unsigned)count), dim3(ALS_THREADS), 0, st, a);
    VPLMC_HIP(hipGetLastError());
    return VPLMC_OK;
}

}  // namespace

int launch_als(hipStream_t st, const vplmc_plan &plan, const SliceDesc *desc, const int32_t *ids_dev,
               const int32_t *gblk_dev, char *gsys, double *e2, const vplmc_params &prm, const int32_t *row_ptr,
               const int32_t *csr_col, const float *csr_val, const int32_t *col_ptr, const int32_t *csc_row,
               const float *csc_val, float *X, float *Xn, float *Y, float *scale, int32_t *row_order, int32_t *col_order,
               int32_t *stats) {
    // with ALS every slice is in its rank bucket's global-memory group (2 b + 1)
    size_t base[9] = {0};
    for (int g = 0; g < 8; ++g) base[g + 1] = base[g] + plan.groups[g].size();
    AlsArgs a;
    a.desc = desc;
    a.seed = prm.seed;
    a.max_iter = prm.max_iter;
    a.mode = ((prm.flags & VPLMC_FIXED_ITERS) ? 1 : 0) | ((prm.flags & VPLMC_GIVEN_INIT) ? 2 : 0);
    a.tol = prm.tol;
    a.lam = prm.lam;
    a.row_ptr_all = row_ptr;
    a.csr_col_all = csr_col;
    a.csr_val_all = csr_val;
    a.col_ptr_all = col_ptr;
    a.csc_row_all = csc_row;
    a.csc_val_all = csc_val;
    a.X_all = X;
    a.Xn_all = Xn;
    a.Y_all = Y;
    a.scale_all = scale;
    a.rord_all = row_order;
    a.cord_all = col_order;
    a.stats_all = stats;
    a.gsys = gsys;
    int rc = VPLMC_OK;
#define VPLMC_ALS_BUCKET(B, Q)                                                      \
    if (!rc) {                                                                      \
        a.ids = ids_dev + base[2 * B + 1];                                          \
        rc = launch_als_q<Q>(st, a, plan, 2 * B + 1, gblk_dev, e2);                 \
    }
    VPLMC_ALS_BUCKET(3, 32)
    VPLMC_ALS_BUCKET(2, 16)
    VPLMC_ALS_BUCKET(1, 8)
    VPLMC_ALS_BUCKET(0, 4)
#undef VPLMC_ALS_BUCKET
    return rc;
}

}  // namespace vplmc
