// Leaf-value refit with the original FP gradients (Sec. 3 eq. (leaf), Sec. 4.2):
// one gather pass over g, h through the leaf-ordered row list, fp64 sums in a
// fixed reduction order (so repeated runs give identical bits); and the score update,
// which shares the layout of finished leaves with it.
#include <type_traits>

#include "refit_device.h"

namespace qgbdt {

// Sums of (g, h) over the pieces of all leaves; one wavefront per unit, four rows per lane in flight.
// After a tree the rows come from the index buffer in which the leaf ended up and go to the caller's list on the way, and (g, h)
// are read as one 8-byte pair from the quantizer's interleaved copy; otherwise the caller's lists are read.
// Bound by the row lists and pairs once per line: see REFIT_EXTRA for the order of the units.
struct RefitTree {  // the tree that has just been grown
    const float2* pairs;
    IdxSet idxs;
    uint32_t id_mask;  // row id of a list's entry
    int32_t* out;
    const RefitUnit* units;
    const int32_t* n_units;
    const int32_t* done;  // 0: the tree is not finished and its leaves are not laid out
};
struct RefitList {  // leaves that the caller lists
    const float *g, *h;
    const int32_t* row_idx;
    LeafList list;
    int2* leaves;  // their units, for the kernel that adds the pieces up
};
template <class SRC>
__global__ __launch_bounds__(256) void refit_partial_kernel(SRC src, int parts, int blocks_per_part, double* __restrict__ partial) {
    constexpr bool TREE = std::is_same<SRC, RefitTree>::value;
    int part, u;
    refit_unit_of(blocks_per_part, part, u);
    RefitUnit un;
    if constexpr (TREE) {
        if (*src.done == 0 || u >= *src.n_units) return;
        un = src.units[u];
    } else {
        if (!find_unit(src.list, parts, u, un)) return;
    }
    const int lane = threadIdx.x & 63;
    const int64_t piece = (int64_t)part * un.n + (u - un.first);
    const int64_t a = min(un.count, piece * un.piece_rows), b = min(un.count, a + un.piece_rows);
    const bool identity = TREE && un.buf == BUF_ORIGINAL;  // a tree that is its root: the list was never stored
    const int32_t* ids;
    if constexpr (TREE) ids = src.idxs.p[un.buf] + un.begin;
    else {
        ids = src.row_idx + un.begin;
        if (piece == 0 && lane == 0) src.leaves[un.leaf] = make_int2(un.first, un.n);
    }
    double G = 0.0, H = 0.0;
    for (int64_t j0 = a; j0 < b; j0 += 256) {
        int32_t r[4];
        float2 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t j = min(j0 + 64 * k + lane, b - 1);
            r[k] = identity ? (int32_t)(un.begin + j) : ids[j];
            if constexpr (TREE) r[k] &= (int32_t)src.id_mask;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if constexpr (TREE) v[k] = src.pairs[r[k]];
            else v[k] = make_float2(src.g[r[k]], src.h[r[k]]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t j = j0 + 64 * k + lane;
            if (j < b) {
                if constexpr (TREE) src.out[un.begin + j] = r[k];
                G += (double)v[k].x;
                H += (double)v[k].y;
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) { G += __shfl_xor(G, o); H += __shfl_xor(H, o); }
    if (lane == 0) reinterpret_cast<double2*>(partial)[(int64_t)parts * un.first + piece] = make_double2(G, H);
}

// One workgroup per leaf: the sums of its pieces.
__global__ __launch_bounds__(256) void refit_final_kernel(const double* __restrict__ partial, int parts,
                                                          const int2* __restrict__ leaves,
                                                          const int32_t* __restrict__ n_leaves_dev,
                                                          const int32_t* __restrict__ done, double* __restrict__ value) {
    const int l = blockIdx.x;
    if (done && *done == 0) return;
    if (n_leaves_dev && l >= *n_leaves_dev) {  // uniform over the workgroup
        if (threadIdx.x == 0) value[l] = 0.0;
        return;
    }
    const int2 lf = leaves[l];
    const double2* p = reinterpret_cast<const double2*>(partial) + (int64_t)parts * lf.x;
    const int n = parts * lf.y;
    double G = 0.0, H = 0.0;
    for (int k = threadIdx.x; k < n; k += blockDim.x) { const double2 v = p[k]; G += v.x; H += v.y; }
    for (int o = 32; o > 0; o >>= 1) { G += __shfl_xor(G, o); H += __shfl_xor(H, o); }
    __shared__ double sg[4], sh[4];
    if ((threadIdx.x & 63) == 0) { sg[threadIdx.x >> 6] = G; sh[threadIdx.x >> 6] = H; }
    __syncthreads();
    if (threadIdx.x == 0) {
        G = ((sg[0] + sg[1]) + sg[2]) + sg[3];
        H = ((sh[0] + sh[1]) + sh[2]) + sh[3];
        value[l] = (H > 0.0) ? -G / H : 0.0;
    }
}

// score[row] += (float)(lr * value[leaf]) for the rows of every leaf, units as above (TREE: those of the tree just grown).
template <bool TREE>
__global__ __launch_bounds__(256) void update_scores_kernel(float* __restrict__ score, const int32_t* __restrict__ row_idx,
                                                            const double* __restrict__ leaf_value,
                                                            const RefitUnit* __restrict__ units, const int32_t* __restrict__ n_units,
                                                            LeafList list, int parts, int blocks_per_part, double lr) {
    int part, u;
    refit_unit_of(blocks_per_part, part, u);
    RefitUnit un;
    if (TREE) {
        if (u >= *n_units) return;
        un = units[u];
    } else if (!find_unit(list, parts, u, un)) return;
    const int lane = threadIdx.x & 63;
    const float d = (float)(lr * leaf_value[un.leaf]);
    const int64_t piece = (int64_t)part * un.n + (u - un.first);
    const int64_t a = min(un.count, piece * un.piece_rows), b = min(un.count, a + un.piece_rows);
    const int32_t* src = row_idx + un.begin;
    for (int64_t j0 = a; j0 < b; j0 += 256) {
        int32_t r[4];
        float v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) r[k] = src[min(j0 + 64 * k + lane, b - 1)];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = score[r[k]];
#pragma unroll
        for (int k = 0; k < 4; ++k)  // every row belongs to exactly one leaf: no two threads touch the same element
            if (j0 + 64 * k + lane < b) score[r[k]] = v[k] + d;
    }
}

struct RefitGrid {
    int parts, blocks_per_part;
    dim3 grid() const { return dim3((unsigned)(parts * blocks_per_part)); }
};
static RefitGrid refit_grid(const qgbdt_ctx* ctx, int n_leaves) {
    RefitGrid r;
    r.parts = refit_parts(ctx->shape.n_rows);
    r.blocks_per_part = (n_leaves + refit_extra(ctx->shape.n_rows) + 3) / 4;
    return r;
}
static const int32_t* units_in_use(const qgbdt_ctx* ctx) { return &ctx->refit_leaves[ctx->shape.max_leaves].x; }

int launch_refit(qgbdt_ctx* ctx, const float* g, const float* h, const int32_t* row_idx, const int64_t* leaf_begin,
                 const int64_t* leaf_count, int n_leaves, double* value_out) {
    if (n_leaves <= 0) return QGBDT_OK;
    const RefitGrid rg = refit_grid(ctx, n_leaves);
    const RefitList src{g, h, row_idx, {leaf_begin, leaf_count, n_leaves, refit_extra(ctx->shape.n_rows)}, ctx->refit_leaves};
    hipLaunchKernelGGL(refit_partial_kernel<RefitList>, rg.grid(), dim3(256), 0, ctx->stream, src, rg.parts, rg.blocks_per_part,
                       ctx->refit_partial);
    hipLaunchKernelGGL(refit_final_kernel, dim3(n_leaves), dim3(256), 0, ctx->stream, ctx->refit_partial, rg.parts,
                       ctx->refit_leaves, nullptr, nullptr, value_out);
    QG_HIP(ctx, hipGetLastError());
    return QGBDT_OK;
}

int launch_gather_refit(qgbdt_ctx* ctx, const IdxSet& idx, uint32_t id_mask, int32_t* row_idx_out, const int32_t* n_leaves_dev, double* value_out) {
    const RefitGrid rg = refit_grid(ctx, ctx->shape.max_leaves);
    const RefitTree src{ctx->ghf, idx, id_mask, row_idx_out, ctx->refit_units, units_in_use(ctx), &ctx->step->done};
    hipLaunchKernelGGL(refit_partial_kernel<RefitTree>, rg.grid(), dim3(256), 0, ctx->stream, src, rg.parts, rg.blocks_per_part,
                       ctx->refit_partial);
    hipLaunchKernelGGL(refit_final_kernel, dim3(ctx->shape.max_leaves), dim3(256), 0, ctx->stream, ctx->refit_partial,
                       rg.parts, ctx->refit_leaves, n_leaves_dev, &ctx->step->done, value_out);
    QG_HIP(ctx, hipGetLastError());
    return QGBDT_OK;
}

int launch_update_scores(qgbdt_ctx* ctx, float* score, const int32_t* row_idx, const int64_t* leaf_begin,
                         const int64_t* leaf_count, const double* leaf_value, int n_leaves, bool laid_out, double lr) {
    if (n_leaves <= 0) return QGBDT_OK;
    const RefitGrid rg = refit_grid(ctx, n_leaves);
    if (laid_out)
        hipLaunchKernelGGL(update_scores_kernel<true>, rg.grid(), dim3(256), 0, ctx->stream, score, row_idx, leaf_value,
                           ctx->refit_units, units_in_use(ctx), LeafList{}, rg.parts, rg.blocks_per_part, lr);
    else
        hipLaunchKernelGGL(update_scores_kernel<false>, rg.grid(), dim3(256), 0, ctx->stream, score, row_idx, leaf_value, nullptr,
                           nullptr, LeafList{leaf_begin, leaf_count, n_leaves, refit_extra(ctx->shape.n_rows)}, rg.parts,
                           rg.blocks_per_part, lr);
    QG_HIP(ctx, hipGetLastError());
    return QGBDT_OK;
}

}  // namespace qgbdt
