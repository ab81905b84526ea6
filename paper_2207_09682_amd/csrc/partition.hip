// Stable row partition of a leaf's index slice (the set I_s of Algorithm 1) by
// bins[row][feature] <= bin.  Two passes: counts of left-going rows per segment (which rows
// they are is kept, as flag bytes here and as bit masks in the batched form), a prefix over
// the segments, then an order-preserving scatter into another buffer.  No inter-workgroup
// waits: signalling between workgroups goes through the memory side on this chip (~1-2 us
// per hop), which a single-pass partition with look-back could not hide.  First the
// stand-alone form behind qgbdt_partition_rows (row ids only), then the batched form of
// grow_tree, which serves all nodes of a round at once and, for narrow rows, also moves the
// bin rows and packed gradients into leaf order.  Trees of up to a few million rows on row
// lists take neither batched pass: their histogram launch counts (CountSource) and
// the split-search launch moves the rows (RowMover).
#include "partition_device.h"

namespace qgbdt {

__device__ __forceinline__ int64_t segment_len(int64_t count, int groups) {
    int64_t seg = (count + groups - 1) / groups;
    return (seg + 255) / 256 * 256;
}

__global__ void fill_i64_kernel(int64_t* p, int64_t v) {
    if (threadIdx.x == 0) *p = v;
}

// Bin of (row, feature) in a row-major matrix of 8-bit (bb = 1) or 16-bit (bb = 2) bins.
__device__ __forceinline__ int bin_at(const uint8_t* __restrict__ bins, int64_t at, int bb) {
    return bb == 2 ? (int)reinterpret_cast<const uint16_t*>(bins)[at] : (int)bins[at];
}

// Rows of a thread whose loads are in flight together, in both stand-alone passes: with one, a row's two dependent loads (and
// the scatter's two barriers per 256 rows) were waited for a dozen and more times in a row by the at most 512 workgroups.
// Bound by the lines of the gathered bins.  The step functions on 3 M x 28 (one partition of all rows): 330 -> 304 us.
constexpr int PART_ROWS = 8;

__global__ __launch_bounds__(256) void part_count_kernel(const uint8_t* __restrict__ bins, int bb, int F,
                                                         const int32_t* __restrict__ src,
                                                         PartWork wk, uint8_t* __restrict__ flags,
                                                         int64_t* __restrict__ counts) {
    const int64_t seg = segment_len(wk.count, gridDim.x);
    const int64_t sbegin = (int64_t)blockIdx.x * seg;
    const int64_t send = min(wk.count, sbegin + seg);
    int cnt = 0;
    for (int64_t t0 = sbegin + threadIdx.x; t0 - threadIdx.x < send; t0 += 256 * PART_ROWS) {
        int64_t row[PART_ROWS];
        int v[PART_ROWS];
#pragma unroll
        for (int u = 0; u < PART_ROWS; ++u) row[u] = src[wk.begin + min(t0 + 256 * u, send - 1)];  // (past the end: the last row again, not counted)
#pragma unroll
        for (int u = 0; u < PART_ROWS; ++u) v[u] = bin_at(bins, row[u] * F + wk.feature, bb);
#pragma unroll
        for (int u = 0; u < PART_ROWS; ++u) {
            const int64_t p = t0 + 256 * u;
            if (p < send) {
                const int fl = v[u] <= wk.bin;
                flags[wk.begin + p] = (uint8_t)fl;
                cnt += fl;
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o);
    __shared__ int sc[4];
    if ((threadIdx.x & 63) == 0) sc[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = (int64_t)sc[0] + sc[1] + sc[2] + sc[3];
}

__global__ __launch_bounds__(256) void part_scatter_kernel(const int32_t* __restrict__ src, int32_t* __restrict__ dst,
                                                           PartWork wk, const uint8_t* __restrict__ flags,
                                                           const int64_t* __restrict__ counts, int64_t* n_left_out) {
    // left rows before this segment, and in total
    int64_t before = 0, total = 0;
    for (int b = threadIdx.x; b < (int)gridDim.x; b += blockDim.x) {
        const int64_t c = counts[b];
        total += c;
        if (b < (int)blockIdx.x) before += c;
    }
    for (int o = 32; o > 0; o >>= 1) { before += __shfl_xor(before, o); total += __shfl_xor(total, o); }
    __shared__ int64_t sb[4], st[4];
    __shared__ int wl[2][4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) { sb[wave] = before; st[wave] = total; }
    __syncthreads();
    before = sb[0] + sb[1] + sb[2] + sb[3];
    total = st[0] + st[1] + st[2] + st[3];
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_left_out = total;

    const int64_t seg = segment_len(wk.count, gridDim.x);
    const int64_t sbegin = (int64_t)blockIdx.x * seg;
    const int64_t send = min(wk.count, sbegin + seg);
    int64_t lpos = wk.begin + before;                      // next left slot
    int64_t rpos = wk.begin + total + (sbegin - before);   // next right slot
    int turn = 0;
    for (int64_t t0 = sbegin; t0 < send; t0 += 256 * PART_ROWS, turn ^= 1) {
        const int w0 = wave * (64 * PART_ROWS) + lane;  // a wavefront's rows are consecutive
        int32_t v[PART_ROWS];
        int fl[PART_ROWS];
#pragma unroll
        for (int u = 0; u < PART_ROWS; ++u) {
            const int64_t p = wk.begin + min(t0 + w0 + 64 * u, send - 1);
            fl[u] = flags[p]; v[u] = src[p];
        }
        unsigned long long m[PART_ROWS];
        int mine = 0;
#pragma unroll
        for (int u = 0; u < PART_ROWS; ++u) {
            m[u] = __ballot(t0 + w0 + 64 * u < send && fl[u]);
            mine += __popcll(m[u]);
        }
        if (lane == 0) wl[turn][wave] = mine;
        __syncthreads();  // (two turns: the next tile's counts go to the other half)
        int lw = 0, ltile = 0;
        for (int k = 0; k < 4; ++k) { const int c = wl[turn][k]; if (k < wave) lw += c; ltile += c; }
#pragma unroll
        for (int u = 0; u < PART_ROWS; ++u) {
            const int rank = lw + __popcll(m[u] & ((1ull << lane) - 1ull));  // left rows of the tile in front of this one
            if (t0 + w0 + 64 * u < send) {
                if (fl[u]) dst[lpos + rank] = v[u];
                else dst[rpos + (w0 + 64 * u - rank)] = v[u];
            }
            lw += __popcll(m[u]);
        }
        const int tile_n = (int)min((int64_t)(256 * PART_ROWS), send - t0);
        lpos += ltile;
        rpos += tile_n - ltile;
    }
}

__global__ void copy_i32_kernel(const int32_t* __restrict__ src, int32_t* __restrict__ dst, int64_t begin,
                                int64_t count) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride)
        dst[begin + i] = src[begin + i];
}

// Stand-alone call: row_idx is reordered in place (through the context's spare buffer).
int run_partition_rows(qgbdt_ctx* ctx, const uint8_t* bins, int32_t* row_idx, int64_t begin, int64_t count,
                       int feature, int bin, int64_t* n_left_out) {
    const PartWork work = {begin, count, feature, bin};
    if (count == 0) {
        hipLaunchKernelGGL(fill_i64_kernel, dim3(1), dim3(64), 0, ctx->stream, n_left_out, (int64_t)0);
        QG_HIP(ctx, hipGetLastError());
        return QGBDT_OK;
    }
    int64_t g = (count + 2047) / 2048;
    if (g > PART_GROUPS) g = PART_GROUPS;
    hipLaunchKernelGGL(part_count_kernel, dim3((unsigned)g), dim3(256), 0, ctx->stream, bins, ctx->shape.bin_bytes,
                       ctx->shape.n_features, row_idx, work, ctx->flags, ctx->part_counts);
    hipLaunchKernelGGL(part_scatter_kernel, dim3((unsigned)g), dim3(256), 0, ctx->stream, row_idx, ctx->idx[0], work,
                       ctx->flags, ctx->part_counts, n_left_out);
    int blocks = (int)((count + 255) / 256);
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(copy_i32_kernel, dim3(blocks), dim3(256), 0, ctx->stream, ctx->idx[0], row_idx, begin, count);
    QG_HIP(ctx, hipGetLastError());
    return QGBDT_OK;
}


// ---- batched partition of the nodes expanded in one round of grow_tree ---------------
//
// Work items are row segments of 256 * R rows (R: part_rows); segment -> (batch entry, segment of that
// node) by binary search over the entries' first-segment numbers.  A wavefront takes 64 * R consecutive rows of
// its segment; which of them go left is one 64-bit mask per 64 rows (128 bytes of masks for 1024 rows instead of a byte
// per row), from which the scatter derives every destination without exchanging anything between wavefronts.

// Left-going rows per segment, as masks and counts; on the way the histogram slots
// that this round's builds accumulate into are cleared.  In ordered mode the rows of a
// node are physically contiguous in its buffer and the bin is read at the row's position;
// otherwise it is gathered from the original matrix through the row id.
// Bound by the gather (a line of the split feature's column, or of the matrix, for one to a few rows at the deep
// levels): all R row ids of a thread, then all its bins are in flight together, and PartOrder lets nodes share the
// lines (both sides there; 10.5 M x 28, bound, 38.9 -> 27.5 us per launch).  Trees whose histogram launch counts the left rows
// (CountSource) do without this pass.
template <int R>
__global__ __launch_bounds__(256) void batch_part_count_kernel(RowSource rows, const uint8_t* __restrict__ bins_t, int64_t n_rows, int ordered,
                                                               int bb, int F, IdxSet idxs,
                                                               const StepState* __restrict__ step,
                                                               const BatchEntry* __restrict__ batch,
                                                               const int32_t* __restrict__ batch_seg,
                                                               unsigned long long* __restrict__ masks,
                                                               int32_t* __restrict__ seg_counts,
                                                               int32_t* __restrict__ super_counts, int64_t* hist_base,
                                                               int64_t hist_words, int shift) {
    constexpr int PART_SEG = 256 * R;
    if (step->done) return;
    const int n_items = step->n_part_items, n_batch = step->n_batch;
    if (n_batch <= 0) return;
    {
        int64_t* z = hist_base + (int64_t)(step->n_slots - n_batch) * hist_words;  // the new slots are the last ones
        const int64_t nz = (int64_t)n_batch * hist_words;
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nz; i += (int64_t)gridDim.x * blockDim.x)
            z[i] = 0;
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    __shared__ int sc[2][4];
    __shared__ int s_start[TABLE_MAX];
    load_batch(batch_seg, n_batch, s_start);
    int turn = 0;
    PartOrder<WaveNodes> order;
    order.start(WaveNodes{lane}, s_start, n_batch, n_items, (int)blockIdx.x, shift);
    for (int at = blockIdx.x; ; at += gridDim.x, turn ^= 1) {
        int node, item;
        if (!order.at(at, node, item)) break;
        const BatchEntry nd = batch[node];
        const int seg = item - nd.seg_start;
        const int sbegin = seg * PART_SEG, n = min(nd.count - sbegin, PART_SEG);  // rows of the segment, inside the node's slice
        const int32_t* src = idxs.p[nd.buf] + nd.begin + sbegin;
        const bool identity = ordered || nd.buf == BUF_ORIGINAL;  // the root's list is the identity
        uint32_t row[R];
        int v[R];
        // (rows past the end: the last one again, not counted; the entries are masked when all are on their way)
        if (identity) {
#pragma unroll
            for (int u = 0; u < R; ++u) row[u] = (uint32_t)(sbegin + min((wave * R + u) * 64 + lane, n - 1));
        } else {
#pragma unroll
            for (int u = 0; u < R; ++u) row[u] = (uint32_t)src[min((wave * R + u) * 64 + lane, n - 1)];
#pragma unroll
            for (int u = 0; u < R; ++u) row[u] &= rows.code.id_mask;
        }
        if (bins_t && !ordered) {
            // with a feature-major copy of the matrix the split feature's column is read: the ascending row
            // ids of a node then fall into few sectors, where the row-major matrix costs one sector per row
            const uint8_t* col = bins_t + (int64_t)nd.feature * n_rows * bb;
#pragma unroll
            for (int u = 0; u < R; ++u) v[u] = bin_at(col, (int64_t)row[u], bb);
        } else {
            const uint8_t* brow = rows.bins[ordered ? nd.buf : BUF_ORIGINAL] + (ordered ? nd.begin * (int64_t)F : 0);
#pragma unroll
            for (int u = 0; u < R; ++u) v[u] = bin_at(brow, (int64_t)row[u] * F + nd.feature, bb);
        }
        int cnt = 0;
        unsigned long long mine = 0ull;  // lane u keeps the wavefront's u-th mask
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const unsigned long long m = __ballot(v[u] <= nd.bin && (wave * R + u) * 64 + lane < n);
            cnt += __popcll(m);
            if (lane == u) mine = m;
        }
        if (lane < R) masks[(int64_t)item * (PART_SEG / 64) + wave * R + lane] = mine;
        if (lane == 0) sc[turn][wave] = cnt;
        __syncthreads();  // (two turns: the next item's counts go to the other half)
        if (threadIdx.x == 0) {
            const int c = sc[turn][0] + sc[turn][1] + sc[turn][2] + sc[turn][3];
            seg_counts[item] = c;
            if (super_counts) atomicAdd(&super_counts[nd.super_start + seg / PART_SUPER], c);
        }
    }
}

// The children of every expanded node and the tables of the histogram and scan kernels, by one workgroup of 256 threads
// while the others move rows: it needs nothing of them but the left counts that the count kernel left behind.
__device__ void child_tables(StepState* step, Node* nodes, const BatchEntry* __restrict__ batch,
                             const int32_t* __restrict__ super_counts, HistEntry* hist_entries, int32_t* hist_counts,
                             ScanPair* pairs, const HistPlan& plan, int super_len, int* s_start, int* s_left, int* s_tmp) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_batch = step->n_batch;
    for (int t = tid; t < n_batch; t += 256) { s_start[t] = batch[t].super_start; s_left[t] = 0; }
    __syncthreads();
    const int last = n_batch - 1;
    const int n_super = s_start[last] + (batch[last].n_seg + super_len - 1) / super_len;
    for (int k = tid; k < n_super; k += 256) {
        int lo = 0, hi = last;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_start[mid] <= k) lo = mid; else hi = mid - 1;
        }
        atomicAdd(&s_left[lo], super_counts[k]);
    }
    __syncthreads();
    // rows of the builds (the smaller children), then their row groups: about max_groups items in total, shared out by size
    int small_total = 0;
    for (int t = tid; t < n_batch; t += 256) {
        const int nl = s_left[t], nr = batch[t].count - nl;
        small_total += min(nl, nr);
    }
    for (int o = 32; o > 0; o >>= 1) small_total += __shfl_xor(small_total, o);
    if (lane == 0) s_tmp[wave] = small_total;
    __syncthreads();
    small_total = s_tmp[0] + s_tmp[1] + s_tmp[2] + s_tmp[3];
    const int target = (int)hist_target_rows(plan, small_total, n_batch);
    int base = 0, big = 0;
    for (int t0 = 0; t0 < n_batch; t0 += 256) {  // (uniform trip count)
        const int t = t0 + tid;
        int nl = 0, nr = 0, groups = 0;
        BatchEntry be;
        if (t < n_batch) {
            be = batch[t];
            nl = s_left[t]; nr = be.count - nl;
            groups = max(1, (min(nl, nr) + target - 1) / target);
            if (groups > plan.search_sums) big = 1;
        }
        const int incl = wave_prefix(groups);
        __syncthreads();
        if (lane == 63) s_tmp[wave] = incl;
        __syncthreads();
        int start = base + incl - groups;
        for (int k = 0; k < wave; ++k) start += s_tmp[k];
        base += s_tmp[0] + s_tmp[1] + s_tmp[2] + s_tmp[3];
        if (t < n_batch) {
            Node* P = &nodes[be.node];
            const int slot = P->slot, child = P->child;
            const int64_t lg = P->best.left_g, lh = P->best.left_h, rg = P->best.right_g, rh = P->best.right_h;
            P->n_left = nl;
            const bool left_small = nl <= nr;
            const int lslot = left_small ? be.new_slot : slot, rslot = left_small ? slot : be.new_slot;
            put_children(nodes, be, child, nl, lg, lh, rg, rh, lslot, rslot);
            HistEntry e;
            e.begin = left_small ? be.begin : be.begin + nl; e.count = left_small ? nl : nr; e.buf = be.child_buf; e.slot = be.new_slot;
            e.item_start = start; e.groups = groups;
            hist_entries[t] = e;
            ScanPair sp;
            sp.slot_a = be.new_slot; sp.slot_b = slot; sp.parent = slot; sp.a_item = left_small ? 0 : 1;
            sp.item_start = start; sp.groups = groups <= plan.search_sums ? groups : 0;
            sp.merged = e.count > (int64_t)groups * plan.single_rows ? 1 : 0; sp.seg_start = 0;
            // (selected number by number: whole records go through scratch memory)
            sp.stat[0].n_rows = left_small ? nl : nr; sp.stat[0].sum_g = left_small ? lg : rg; sp.stat[0].sum_h = left_small ? lh : rh;
            sp.stat[1].n_rows = left_small ? nr : nl; sp.stat[1].sum_g = left_small ? rg : lg; sp.stat[1].sum_h = left_small ? rh : lh;
            pairs[t] = sp;
        }
    }
    big = __syncthreads_or(big);
    if (tid == 0) { hist_counts[0] = n_batch; hist_counts[1] = base; hist_counts[2] = big; hist_counts[3] = (int32_t)small_total; }
}

// Order-preserving scatter of every segment into the children's buffer.  The left rows in front of a segment are the sum
// of the node's super counts (SUPER segments each) and of the segment counts in front of it inside its super group: every wavefront adds them
// up for itself (DPP sums), reads the segment's masks and knows where each of its rows goes, so no wavefront waits for
// another.  In ordered mode (MODE 2) the bin rows then move as dwords, eight independent loads per thread in flight,
// coalesced on the reading side and in two compacted streams on the writing side; the packed gradients move with the row ids.
// The first workgroup builds the next kernels' tables meanwhile (child_tables), which was a launch of its own between the
// two passes: 12.2 us per round on 10.5 M x 28.  Bound by the copy: 15.3 us per launch on 10.5 M x 28 (entries of 4 bytes),
// 27 us on 20 M x 200 (row ids and packed gradients).
// Bin rows that come from beyond the caches (MODE 2 with the counters): five wavefronts per SIMD, not the six that the registers allow, copy 14 M x 32 in 155
// instead of 161 us per launch (trees of 14 M x 32 3738 / 3660 us, 12 M x 16 2148 / 2133, 7 M x 28 1570 / 1567; smaller ones, without the counters, 3 M x 20 1060 / 1078).
template <int MODE, int R, int SUPER>  // 0: row ids, 1: row ids and packed gradients, 2: those and the bin rows (ordered mode)
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, MODE == 2 && SUPER > 1 ? 5 : 8))) void batch_part_scatter_kernel(RowSource rows, RowDest out, int F, IdxSet idxs,
                                                                 StepState* step, const BatchEntry* __restrict__ batch,
                                                                 const int32_t* __restrict__ batch_seg, Node* nodes,
                                                                 const unsigned long long* __restrict__ masks,
                                                                 const int32_t* __restrict__ seg_counts,
                                                                 const int32_t* __restrict__ super_counts,
                                                                 HistEntry* hist_entries, int32_t* hist_counts,
                                                                 ScanPair* pairs, HistPlan plan) {
    constexpr int PART_SEG = 256 * R;
    if (step->done) return;
    __shared__ int s_start[TABLE_MAX];
    __shared__ int s_dpos[MODE == 2 && PART_SEG > TABLE_MAX + 8 ? PART_SEG : TABLE_MAX + 8];  // (also child_tables' LDS)
    if (blockIdx.x == 0) {
        child_tables(step, nodes, batch, super_counts, hist_entries, hist_counts, pairs, plan, SUPER, s_start, s_dpos, s_dpos + TABLE_MAX);
        return;
    }
    const int n_items = step->n_part_items, n_batch = step->n_batch;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int dpr = F / 4;
    load_batch(batch_seg, n_batch, s_start);
    // Segments are taken from the last to the first: in ordered mode the count kernel has just streamed the same rows front to back, so the
    // tail of that stream is what the memory-side cache still holds.  (Row lists, counted by PartOrder, take the same time either
    // way: 10.5 M x 28 16.1 / 16.2 us per launch, 5 M x 200 17.5 / 17.5, 8 M x 28 not bound 14.5 / 14.8.)
    for (int item = n_items - (int)blockIdx.x; item >= 0; item -= (int)gridDim.x - 1) {
        const BatchEntry nd = batch[find_start(s_start, n_batch, item)];
        scatter_wave<MODE, R, SUPER>(rows, out.gh, idxs, nd, item, wave, lane, masks, seg_counts, super_counts, s_dpos);
        if (MODE == 2) {
            const int sbegin = (item - nd.seg_start) * PART_SEG, n = min(nd.count - sbegin, PART_SEG);
            const uint8_t* bsrc = rows.bins[nd.buf] + (nd.begin + sbegin) * (int64_t)F;
            uint8_t* bdst = out.bins[nd.child_buf] + nd.begin * (int64_t)F;
            __syncthreads();
            const uint32_t* s32 = reinterpret_cast<const uint32_t*>(bsrc);
            const int n_dw = n * dpr;
            for (int e0 = threadIdx.x; e0 < n_dw; e0 += 8 * 256) {
                uint32_t v8[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int e = e0 + u * 256;
                    v8[u] = e < n_dw ? s32[e] : 0u;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int e = e0 + u * 256;
                    if (e < n_dw) {
                        const int r = e / dpr, q = e - r * dpr;
                        reinterpret_cast<uint32_t*>(bdst + (int64_t)s_dpos[r] * F)[q] = v8[u];
                    }
                }
            }
            __syncthreads();  // s_dpos is reused by the next item
        }
    }
}

static int batch_part_grid(const qgbdt_ctx* ctx) {
    int64_t g = ctx->max_seg;
    if (g > 2048) g = 2048;
    if (g < 1) g = 1;
    return (int)g;
}

static IdxSet idx_set(const qgbdt_ctx* ctx) {
    IdxSet s;
    for (int b = 0; b < ROW_BUFS; ++b) s.p[b] = ctx->idx[b];
    s.p[BUF_ORIGINAL] = ctx->idx[0];
    return s;
}

namespace {
struct HostNodes {  // WaveNodes, one node after the other
    template <class F>
    int sum(int n, F f) const {
        int c = 0;
        for (int j = 0; j < n; ++j) c += f(j);
        return c;
    }
    int last_start(const int* starts, int n, int at) const {
        int c = 0;
        while (c < n && starts[c] <= at) ++c;
        return c - 1;
    }
    template <class F>
    bool find(int n, F share, int& at, int& node, int& from) const {
        for (node = 0; node < n; ++node) {
            const int k = share(node, from);
            if (at < k) return true;
            at -= k;
        }
        return false;
    }
};
}  // namespace

int64_t order_of_segments(const qgbdt_shape& s, bool bound, const int32_t* starts, int n_nodes, int n_segs, int block, int grid, int32_t* out, int64_t room) {
    PartOrder<HostNodes> order;
    order.start(HostNodes{}, starts, n_nodes, n_segs, block, order_shift(s.n_rows, bound));
    int64_t n = 0;
    for (int at = block, node, item; order.at(at, node, item); at += grid, ++n)
        if (n < room) { out[2 * n] = node; out[2 * n + 1] = item; }
    return n;
}

int launch_batch_partition_count(qgbdt_ctx* ctx, const RowSource& rows, const uint8_t* bins_t, bool ordered) {
    const int64_t W = (int64_t)ctx->shape.n_features * ctx->shape.n_bins;
#define QG_COUNT(R_)                                                                                                   \
    hipLaunchKernelGGL(batch_part_count_kernel<R_>, dim3((batch_part_grid(ctx) + 7) / 8 * 8), dim3(256), 0, ctx->stream, rows, bins_t, \
                       ctx->shape.n_rows, ordered ? 1 : 0, ctx->shape.bin_bytes, ctx->shape.n_features, idx_set(ctx),  \
                       ctx->step, ctx->batch, ctx->batch_seg, ctx->part_masks, ctx->seg_counts, supers, \
                       ctx->hist_pool, W, ordered ? 0 : order_shift(ctx->shape.n_rows, bins_t != nullptr))
    int32_t* const supers = ctx->seg_supers ? ctx->super_counts : nullptr;
    if (ctx->seg_rows == 256 * 8) QG_COUNT(8); else QG_COUNT(2);
#undef QG_COUNT
    QG_HIP(ctx, hipGetLastError());
    return QGBDT_OK;
}

int launch_batch_partition_scatter(qgbdt_ctx* ctx, const RowSource& rows, bool ordered, const HistPlan& plan) {
    RowDest out;
    for (int b = 0; b < COPY_BUFS; ++b) out.bins[b] = ctx->obins[b];
    for (int b = 0; b < ROW_BUFS; ++b) out.gh[b] = ctx->ogh[b];
    const int32_t* const sums = ctx->seg_supers ? ctx->super_counts : ctx->seg_counts;
#define QG_SCATTER_R(MODE_, R_, S_)                                                                                    \
    hipLaunchKernelGGL((batch_part_scatter_kernel<MODE_, R_, S_>), dim3(batch_part_grid(ctx) + 1), dim3(256), 0, ctx->stream,     \
                       rows, out, ctx->shape.n_features, idx_set(ctx), ctx->step, ctx->batch, ctx->batch_seg,           \
                       ctx->nodes, ctx->part_masks, ctx->seg_counts, sums, ctx->hist_entries,                           \
                       ctx->hist_counts, ctx->scan_pairs, plan)
#define QG_SCATTER(MODE_)                                                  \
    do {                                                                   \
        if (ctx->seg_supers) QG_SCATTER_R(MODE_, 8, PART_SUPER);           \
        else if (ctx->seg_rows == 256 * 8) QG_SCATTER_R(MODE_, 8, 1);      \
        else QG_SCATTER_R(MODE_, 2, 1);                                    \
    } while (0)
    if (ordered) QG_SCATTER(2);
    else if (rows.gh_pos) QG_SCATTER(1);
    else QG_SCATTER(0);
#undef QG_SCATTER
#undef QG_SCATTER_R
    QG_HIP(ctx, hipGetLastError());
    return QGBDT_OK;
}

// Feature-major copy of a row-major bin matrix: out[f][row] = in[row][f], 32 x 32 tiles through LDS
// so that both sides are accessed along their contiguous direction.
template <typename T>
__global__ __launch_bounds__(256) void transpose_bins_kernel(const T* __restrict__ in, T* __restrict__ out, int64_t N, int F) {
    __shared__ T tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
    const int64_t tiles_r = (N + 31) / 32;
    const int tiles_f = (F + 31) / 32;
    for (int64_t t = blockIdx.x; t < tiles_r * tiles_f; t += gridDim.x) {
        const int64_t r0 = (t / tiles_f) * 32;
        const int f0 = (int)(t % tiles_f) * 32;
        __syncthreads();
        for (int k = ty; k < 32; k += 8)
            if (r0 + k < N && f0 + tx < F) tile[k][tx] = in[(r0 + k) * F + f0 + tx];
        __syncthreads();
        for (int k = ty; k < 32; k += 8)
            if (f0 + k < F && r0 + tx < N) out[(int64_t)(f0 + k) * N + r0 + tx] = tile[tx][k];
    }
}

// The same for 8-bit bins when both the row count and the feature count are multiples of 4: 64 x 64 tiles, a
// dword (four features of a row) per load and a dword (four rows of a feature) per store.
__global__ __launch_bounds__(256) void transpose_bins4_kernel(const uint8_t* __restrict__ in, uint8_t* __restrict__ out,
                                                              int64_t N, int F) {
    __shared__ uint8_t tile[64][68];  // [row][feature]; pitch 68 keeps the dword stores of a row aligned
    const int c = threadIdx.x & 15, r = threadIdx.x >> 4;  // 16 dword columns x 16 rows per pass
    const int64_t tiles_r = (N + 63) / 64;
    const int tiles_f = (F + 63) / 64;
    for (int64_t t = blockIdx.x; t < tiles_r * tiles_f; t += gridDim.x) {
        const int64_t r0 = (t / tiles_f) * 64;
        const int f0 = (int)(t % tiles_f) * 64;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int rr = r + 16 * k;
            uint32_t v = 0u;
            if (r0 + rr < N && f0 + 4 * c < F) v = *reinterpret_cast<const uint32_t*>(in + (r0 + rr) * F + f0 + 4 * c);
            *reinterpret_cast<uint32_t*>(&tile[rr][4 * c]) = v;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int ff = r + 16 * k;  // feature of the tile; c: group of four rows
            if (f0 + ff < F && r0 + 4 * c < N) {
                const uint32_t v = (uint32_t)tile[4 * c][ff] | ((uint32_t)tile[4 * c + 1][ff] << 8) |
                                   ((uint32_t)tile[4 * c + 2][ff] << 16) | ((uint32_t)tile[4 * c + 3][ff] << 24);
                *reinterpret_cast<uint32_t*>(out + (int64_t)(f0 + ff) * N + r0 + 4 * c) = v;
            }
        }
    }
}

// Copy of a matrix of 8-byte units at a larger pitch; a workgroup takes consecutive units.
__global__ __launch_bounds__(256) void pad_bins_kernel(const uint8_t* __restrict__ in, uint2* __restrict__ out, int64_t n_units, int row_units, int pitch_units,
                                                       int64_t per_block) {
    const int64_t first = (int64_t)blockIdx.x * per_block, last = min(n_units, first + per_block);
    int64_t i = first + threadIdx.x;
    if (i >= last) return;
    int64_t row = i / row_units;
    int c = (int)(i - row * row_units);
    const int drow = 256 / row_units, dc = 256 - drow * row_units;
    for (; i < last; i += 256) {
        uint2 v;
        __builtin_memcpy(&v, in + 8 * i, 8);  // (the caller's matrix may begin anywhere)
        out[row * pitch_units + c] = v;
        row += drow; c += dc;
        if (c >= row_units) { c -= row_units; ++row; }
    }
}

int launch_pad_bins(qgbdt_ctx* ctx, const void* bins, uint8_t* out, int pitch) {
    const int64_t n = ctx->shape.n_rows * (ctx->shape.n_features / 8), per = (n + 8191) / 8192;
    hipLaunchKernelGGL(pad_bins_kernel, dim3((unsigned)((n + per - 1) / per)), dim3(256), 0, ctx->stream, static_cast<const uint8_t*>(bins),
                       reinterpret_cast<uint2*>(out), n, ctx->shape.n_features / 8, pitch / 8, per);
    QG_HIP(ctx, hipGetLastError());
    return QGBDT_OK;
}

// Most frequent bin of every feature, from a strided sample of at most 65536 rows of the feature-major copy (the
// choice only steers which bin the histogram kernels leave out; any bin would be correct).  mfb[f] = that bin when
// it holds at least half of the sampled rows, else 0xffff.  One workgroup per feature.
template <typename T>
__global__ __launch_bounds__(256) void frequent_bins_kernel(const T* __restrict__ bins_t, int64_t N, int nb,
                                                            uint16_t* __restrict__ mfb) {
    __shared__ int cnt[1024];
    __shared__ int s_best[4], s_bin[4];
    const int f = blockIdx.x;
    for (int b = threadIdx.x; b < 1024; b += blockDim.x) cnt[b] = 0;
    __syncthreads();
    const int64_t stride = N > 65536 ? N / 65536 : 1;
    const int64_t n_s = N > 65536 ? 65536 : N;
    const T* col = bins_t + (int64_t)f * N;
    for (int64_t j = threadIdx.x; j < n_s; j += blockDim.x) {
        const int v = (int)col[j * stride];
        // lanes with equal values are counted by one of them: same-address LDS atomics serialize
        const unsigned long long active = __ballot(1);
        unsigned long long rest = active;
        const int lane = threadIdx.x & 63;
        while (rest) {
            const int lead = __ffsll((long long)rest) - 1;
            const int lv = __shfl(v, lead);
            const unsigned long long same = __ballot(v == lv) & rest;
            if (lane == lead) atomicAdd(&cnt[lv], __popcll(same));
            rest &= ~same;
        }
    }
    __syncthreads();
    int best = -1, bin = 0;
    for (int b = threadIdx.x; b < nb; b += blockDim.x)
        if (cnt[b] > best) { best = cnt[b]; bin = b; }
    for (int o = 32; o > 0; o >>= 1) {
        const int ob = __shfl_xor(best, o), obin = __shfl_xor(bin, o);
        if (ob > best || (ob == best && obin < bin)) { best = ob; bin = obin; }
    }
    if ((threadIdx.x & 63) == 0) { s_best[threadIdx.x >> 6] = best; s_bin[threadIdx.x >> 6] = bin; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < 4; ++k)
            if (s_best[k] > best || (s_best[k] == best && s_bin[k] < bin)) { best = s_best[k]; bin = s_bin[k]; }
        mfb[f] = (2 * (int64_t)best >= n_s) ? (uint16_t)bin : (uint16_t)0xffff;
    }
}

int launch_frequent_bins(qgbdt_ctx* ctx, const void* bins_t, uint16_t* mfb) {
    const int64_t N = ctx->shape.n_rows;
    const int F = ctx->shape.n_features, nb = ctx->shape.n_bins;
    if (ctx->shape.bin_bytes == 2)
        hipLaunchKernelGGL(frequent_bins_kernel<uint16_t>, dim3(F), dim3(256), 0, ctx->stream,
                           static_cast<const uint16_t*>(bins_t), N, nb, mfb);
    else
        hipLaunchKernelGGL(frequent_bins_kernel<uint8_t>, dim3(F), dim3(256), 0, ctx->stream,
                           static_cast<const uint8_t*>(bins_t), N, nb, mfb);
    QG_HIP(ctx, hipGetLastError());
    return QGBDT_OK;
}

// Completes a stand-alone histogram whose kernels left out the most frequent bins: the entry of feature f's
// bin mfb[f] becomes the build's totals minus the feature's other entries.  totals: (sum g~, sum h~).
__global__ __launch_bounds__(256) void fix_frequent_bins_kernel(int64_t* hist, const int64_t* __restrict__ totals,
                                                                const uint16_t* __restrict__ mfb, int F, int nb) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= F) return;
    const int mb = mfb[f];
    if (mb == 0xffff) return;
    int64_t all = 0;
    for (int b = 0; b < nb; ++b) all += hist[(int64_t)b * F + f];
    hist[(int64_t)mb * F + f] += (totals[0] * 4294967296LL + totals[1]) - all;
}

int launch_fix_frequent_bins(qgbdt_ctx* ctx, int64_t* hist, const int64_t* totals, const uint16_t* mfb) {
    const int F = ctx->shape.n_features;
    hipLaunchKernelGGL(fix_frequent_bins_kernel, dim3((F + 255) / 256), dim3(256), 0, ctx->stream, hist, totals, mfb, F,
                       ctx->shape.n_bins);
    QG_HIP(ctx, hipGetLastError());
    return QGBDT_OK;
}

int launch_transpose_bins(qgbdt_ctx* ctx, const void* bins, void* out) {
    const int64_t N = ctx->shape.n_rows;
    const int F = ctx->shape.n_features;
    if (ctx->shape.bin_bytes == 1 && N % 4 == 0 && F % 4 == 0 && (((uintptr_t)bins | (uintptr_t)out) & 3) == 0) {
        const int64_t tiles4 = ((N + 63) / 64) * ((F + 63) / 64);
        hipLaunchKernelGGL(transpose_bins4_kernel, dim3((unsigned)(tiles4 < 65536 ? tiles4 : 65536)), dim3(256), 0,
                           ctx->stream, static_cast<const uint8_t*>(bins), static_cast<uint8_t*>(out), N, F);
        QG_HIP(ctx, hipGetLastError());
        return QGBDT_OK;
    }
    int64_t tiles = ((N + 31) / 32) * ((F + 31) / 32);
    const int grid = (int)(tiles < 65536 ? tiles : 65536);
    if (ctx->shape.bin_bytes == 2)
        hipLaunchKernelGGL(transpose_bins_kernel<uint16_t>, dim3(grid), dim3(256), 0, ctx->stream,
                           static_cast<const uint16_t*>(bins), static_cast<uint16_t*>(out), N, F);
    else
        hipLaunchKernelGGL(transpose_bins_kernel<uint8_t>, dim3(grid), dim3(256), 0, ctx->stream,
                           static_cast<const uint8_t*>(bins), static_cast<uint8_t*>(out), N, F);
    QG_HIP(ctx, hipGetLastError());
    return QGBDT_OK;
}

}  // namespace qgbdt
