// The loss derivatives g_i, h_i of the current predictions, which start a boosting iteration on
// the device (Sec. 3): binary cross-entropy (HBM-bound streaming) and lambdarank.
#include "common.h"

namespace qgbdt {

// p = 1 / (1 + exp(-s)) in fp64 from the fp32 score, g = p - y, h = p (1 - p), each rounded
// once to fp32: 16 bytes of traffic per row hide the fp64 arithmetic.
__device__ __forceinline__ void logistic_one(float s, float y, float& g, float& h) {
    const double p = 1.0 / (1.0 + exp(-(double)s));
    g = (float)(p - (double)y);
    h = (float)(p * (1.0 - p));
}

template <bool VEC>
__global__ __launch_bounds__(256) void logistic_grad_kernel(const float* __restrict__ score,
                                                            const float* __restrict__ label, int64_t n,
                                                            float* __restrict__ g, float* __restrict__ h) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (VEC) {  // all four arrays 16-byte aligned
        const int64_t n4 = n >> 2;
        for (int64_t i = t0; i < n4; i += stride) {
            const float4 s = reinterpret_cast<const float4*>(score)[i], y = reinterpret_cast<const float4*>(label)[i];
            float4 go, ho;
            logistic_one(s.x, y.x, go.x, ho.x); logistic_one(s.y, y.y, go.y, ho.y);
            logistic_one(s.z, y.z, go.z, ho.z); logistic_one(s.w, y.w, go.w, ho.w);
            reinterpret_cast<float4*>(g)[i] = go;
            reinterpret_cast<float4*>(h)[i] = ho;
        }
        const int64_t r = (n4 << 2) + t0;
        if (r < n) logistic_one(score[r], label[r], g[r], h[r]);
    } else {
        for (int64_t i = t0; i < n; i += stride) logistic_one(score[i], label[i], g[i], h[i]);
    }
}

// Pairwise ranking loss with NDCG weights (lambdarank) over queries of `group` consecutive rows.  For a pair (a, b) of a
// query with rel_a > rel_b:
//   rho = 1 / (1 + exp(s_a - s_b)),  w = |gain_a - gain_b| |disc_a - disc_b| / maxDCG,
//   g_a -= rho w, g_b += rho w, h_a += rho (1 - rho) w, h_b += rho (1 - rho) w;  fp64, rounded once.
// One thread per document, as many whole queries per workgroup as fill its wavefronts; a thread walks all documents of
// its query twice (ranks, then pairs), so its sums need no atomics and have a fixed order.
// Bound by the vector ALU (group^2 fp64 pair terms per query against 16 bytes per row), so the steps of a pair are few:
//  * with F = exp(c - s), c the middle of the query's score range, rho = F_a t and 1 - rho = F_b t for t = 1 / (F_a + F_b):
//    one exp per document, and t serves both derivatives: g takes F_x w t, h takes F_k F_j w t^2 (F_k after the loop);
//  * four pairs share one reciprocal, that of the product of their sums: the hardware's estimate and one third-order
//    step cost 7 instruction times, shared by four, and the products 9 (15 instruction times per pair
//    in all, 26 before).  The product of four sums, and t^2 times a weight, must stay finite and normal: queries with a
//    score range of 340 or more, or gains beyond 1e100, take one reciprocal per pair and the factors F_a t and F_b t
//    themselves, which lie between 0 and 1 (2 M rows, queries of 100, scores in +-200: 407 us by the direct form, 157 us so;
//    the four pairs' form takes 130); from 690 on exp(c - s) is no longer safe, and every pair takes its own exp and
//    division (the direct form);
//  * ranks are counted over 64-bit keys (order of the value, then of the position): one comparison and one add-with-
//    carry per partner and rank instead of two comparisons in fp64, one of positions and the logic between them;
//  * discounts come from a table made once per workgroup (log2 and a division per rank instead of two per document).
// 20 M rows, queries of 100: 2.7 -> 1.45 ms (lanes in use 78 -> 98 %); derivatives that are not the 80-bit result rounded, scores of
// deviation 20: 61 -> 19 of 80,000.
__device__ __forceinline__ double recip(double d) {
    const double y = __builtin_amdgcn_rcp(d);  // relative error below 2^-23: its third power is far below fp64's
    const double e = fma(-d, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// Unsigned key that orders as the float does (-0 like +0), ties by position: the earlier one is larger.
__device__ __forceinline__ unsigned long long rank_key(float v, int k) {
    uint32_t b = __float_as_uint(v);
    if ((b << 1) == 0u) b = 0u;
    b = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
    return ((unsigned long long)b << 32) | (uint32_t)~k;
}

constexpr int RANK_QUERIES_MAX = 32;  // queries per workgroup

// Documents per query in LDS: multiples of 4 (16-byte reads of two values), an odd number of them, so that the queries of
// a wavefront read from different banks.
__host__ __device__ __forceinline__ int rank_pitch(int group) { return (((group + 3) >> 2) | 1) << 2; }

__global__ __launch_bounds__(1024) void lambdarank_grad_kernel(const float* __restrict__ score,
                                                               const float* __restrict__ label, int64_t n, int group,
                                                               int queries, float* __restrict__ g, float* __restrict__ h) {
    extern __shared__ __align__(16) double lr_lds[];
    const int pitch = rank_pitch(group), slots = queries * pitch;
    ulonglong2* const keys = reinterpret_cast<ulonglong2*>(lr_lds);  // [slots] keys of score and relevance
    double* const gain = lr_lds + 2 * slots;                         // [slots]
    double* const disc = gain + slots;                               // [slots]
    double* const fac = disc + slots;                                // [slots] exp(c - s)
    double* const part = fac + slots;                                // [slots] terms of the ideal DCG
    double* const table = part + slots;                              // [group] discount of a rank
    __shared__ float s_max[RANK_QUERIES_MAX], s_min[RANK_QUERIES_MAX];
    __shared__ double s_dcg[RANK_QUERIES_MAX];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), n_waves = blockDim.x >> 6;
    const int per_batch = queries * group;
    const int q = tid / group, k = tid - q * group, at = q * pitch;
    const int64_t b0 = (int64_t)blockIdx.x * per_batch, q0 = b0 + (int64_t)q * group;  // first row of the workgroup, of the thread's query
    const bool on = tid < per_batch && q0 + k < n;
    const int m = on ? (int)min((int64_t)group, n - q0) : 0;
    float sk = 0.0f, rk = 0.0f;
    if (on) { sk = score[q0 + k]; rk = label[q0 + k]; }
    for (int i = tid; i < group; i += blockDim.x) table[i] = 1.0 / log2((double)i + 2.0);
    const unsigned long long ks = rank_key(sk, k), kr = rank_key(rk, k);
    if (on) keys[at + k] = make_ulonglong2(ks, kr);
    __syncthreads();
    double gk = 0.0, dk = 0.0;
    if (on) {
        int rank = 0, irank = 0;
#pragma unroll 4
        for (int j = 0; j < m; ++j) {
            const ulonglong2 kj = keys[at + j];
            rank += kj.x > ks ? 1 : 0;
            irank += kj.y > kr ? 1 : 0;
        }
        gk = exp2((double)rk) - 1.0;
        dk = table[rank];
        gain[at + k] = gk; disc[at + k] = dk; part[at + k] = gk * table[irank];
        if (rank == 0) s_max[q] = sk;  // (a NaN is first or last by its key)
        if (rank == m - 1) s_min[q] = sk;
    }
    __syncthreads();
    for (int p = wave; p < queries; p += n_waves) {  // a wavefront adds up a query's ideal DCG
        const int64_t p0 = b0 + (int64_t)p * group;
        double sum = 0.0;
        for (int j = lane; j < group && p0 + j < n; j += 64) sum += part[p * pitch + j];
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
        if (lane == 0) s_dcg[p] = sum;
    }
    double smax = 0.0, smin = 0.0, fk = 0.0;
    if (on) {
        smax = (double)s_max[q]; smin = (double)s_min[q];
        fk = exp(0.5 * (smax + smin) - (double)sk);
        fac[at + k] = fk;
    }
    __syncthreads();
    if (!on) return;
    const double max_dcg = s_dcg[q];
    double G = 0.0, H = 0.0;
    if (max_dcg > 0.0) {
        const bool nan_score = smax != smax || smin != smin;
        if (nan_score || ((smax - smin) < 340.0 && max_dcg < 1.0e100)) {  // (a NaN reaches every document of its query)
            auto pair = [&](double gj, double dj, double fj, double t) {
                const double dg = gk - gj;
                const double u = dg * fabs(dk - dj) * t;  // 0 for equal relevance
                G = fma(-(dg > 0.0 ? fk : fj), u, G);
                H = fma(fabs(u) * t, fj, H);
            };
            const double2* const g2 = reinterpret_cast<const double2*>(gain + at);
            const double2* const d2 = reinterpret_cast<const double2*>(disc + at);
            const double2* const f2 = reinterpret_cast<const double2*>(fac + at);
            int j = 0;
            for (; j + 4 <= m; j += 4) {
                const double2 fa = f2[j >> 1], fb = f2[(j >> 1) + 1], ga = g2[j >> 1], gb = g2[(j >> 1) + 1];
                const double2 da = d2[j >> 1], db = d2[(j >> 1) + 1];
                const double s0 = fk + fa.x, s1 = fk + fa.y, s2 = fk + fb.x, s3 = fk + fb.y;
                const double s01 = s0 * s1, s23 = s2 * s3, r = recip(s01 * s23), r01 = r * s23, r23 = r * s01;
                pair(ga.x, da.x, fa.x, r01 * s1);
                pair(ga.y, da.y, fa.y, r01 * s0);
                pair(gb.x, db.x, fb.x, r23 * s3);
                pair(gb.y, db.y, fb.y, r23 * s2);
            }
            for (; j < m; ++j) pair(gain[at + j], disc[at + j], fac[at + j], recip(fk + fac[at + j]));
            H *= fk;
        } else if ((smax - smin) < 690.0) {
#pragma unroll 2
            for (int j = 0; j < m; ++j) {
                const double fj = fac[at + j], t = recip(fk + fj), a = fk * t, b = fj * t;
                const double dg = gk - gain[at + j], u = dg * fabs(dk - disc[at + j]);
                G = fma(-(dg > 0.0 ? a : b), u, G);
                H = fma(a * b, fabs(u), H);
            }
        } else {
            const double sd = (double)sk;
            for (int j = 0; j < m; ++j) {
                const double gj = gain[at + j], sj = (double)score[q0 + j];
                if (gj == gk) continue;
                const bool up = gk > gj;
                const double w = fabs(gk - gj) * fabs(dk - disc[at + j]);
                const double rho = 1.0 / (1.0 + exp(up ? sd - sj : sj - sd));
                G += up ? -rho * w : rho * w;
                H += rho * (1.0 - rho) * w;
            }
        }
        G /= max_dcg; H /= max_dcg;
    }
    g[q0 + k] = (float)G;
    h[q0 + k] = (float)H;
}

// Queries per workgroup: what costs the busiest compute unit the fewest wavefronts -- whole wavefronts per workgroup times
// its workgroups -- with at most 512 threads, or one query (20 M rows of queries of 100: five in 512 threads, 98 % of the
// lanes in use, against 78 % for one in 128; 2000 queries: four in 448 threads).
static int rank_queries(int64_t n_queries, int group) {
    int best = 1;
    int64_t best_cost = INT64_MAX;
    for (int q = 1; q <= RANK_QUERIES_MAX && (q == 1 || q * group <= 512); ++q) {
        const int64_t batches = (n_queries + q - 1) / q, cost = (batches + 255) / 256 * ((q * group + 63) / 64);
        if (cost < best_cost) { best_cost = cost; best = q; }
    }
    return best;
}

int launch_lambdarank_gradients(qgbdt_ctx* ctx, const float* score, const float* label, int64_t n, int group,
                                float* g, float* h) {
    if (n <= 0) return QGBDT_OK;
    const int64_t n_queries = (n + group - 1) / group;
    const int queries = rank_queries(n_queries, group);
    const int threads = (queries * group + 63) / 64 * 64;
    const size_t lds = sizeof(double) * (6 * (size_t)queries * rank_pitch(group) + (size_t)group);
    // a launch holds fewer than 2^32 work-items (queries of one row fill half of a wavefront): 2^31 at most, then the next one
    const int64_t per_batch = (int64_t)queries * group, most = ((int64_t)1 << 31) / threads * per_batch;
    for (int64_t first = 0; first < n; first += most) {
        const int64_t rows = n - first < most ? n - first : most;
        hipLaunchKernelGGL(lambdarank_grad_kernel, dim3((unsigned)((rows + per_batch - 1) / per_batch)), dim3(threads), lds,
                           ctx->stream, score + first, label + first, rows, group, queries, g + first, h + first);
    }
    QG_HIP(ctx, hipGetLastError());
    return QGBDT_OK;
}

int launch_logistic_gradients(qgbdt_ctx* ctx, const float* score, const float* label, int64_t n, float* g, float* h) {
    if (n <= 0) return QGBDT_OK;
    const bool vec = ((((uintptr_t)score | (uintptr_t)label | (uintptr_t)g | (uintptr_t)h) & 15) == 0);
    int blocks = (int)(((vec ? (n + 3) / 4 : n) + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    if (vec) hipLaunchKernelGGL(logistic_grad_kernel<true>, dim3(blocks), dim3(256), 0, ctx->stream, score, label, n, g, h);
    else hipLaunchKernelGGL(logistic_grad_kernel<false>, dim3(blocks), dim3(256), 0, ctx->stream, score, label, n, g, h);
    QG_HIP(ctx, hipGetLastError());
    return QGBDT_OK;
}

}  // namespace qgbdt
