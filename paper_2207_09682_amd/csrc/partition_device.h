// Device parts of the batched partition shared by its own kernels and the split search, which moves the rows of
// a round where the histogram launch has counted them.
#pragma once
#include "split_device.h"

namespace qgbdt {

// (The entries' first segments are copied into LDS once per workgroup and searched there: through global memory the
// search is a chain of dependent loads per segment.)
__device__ __forceinline__ void load_batch(const int32_t* __restrict__ batch_seg, int n_batch, int* s_start) {
    for (int t = threadIdx.x; t < n_batch; t += blockDim.x) s_start[t] = batch_seg[t];
    __syncthreads();
}

// The order in which a round's segments are counted.  A node's rows are spread over all the matrix, in ascending order, so the s-th of its
// n segments lies about s / n of the way through it, and nodes that split by the same feature read the same lines of its column (without
// the feature-major copy: all nodes the same lines of the matrix).  Every XCD therefore takes an eighth of each node, the same one,
// and goes through the eighths of all nodes side by side, in 2^shift / 8 steps: a line is then fetched by the first node and
// found in the XCD's L2 by the others.  (Workgroup ids go round-robin to the XCDs.)
// Per launch against segments in the order of the nodes, with 1 / 2 / 4 / 8 steps: 2 M x 40 of 16-bit bins 11.8 -> 9.8 / 10.0 / 10.3 / 10.4 us, 4 M x 28 15.0 -> 11.6 /
// 11.7 / 12.5 / 13.0, 8 M x 28 31.0 -> 24.6 / 23.6 / 22.6 / 22.9, 10.5 M x 28 38.9 -> 30.0 / 28.5 / 27.5 / 27.5, 5 M x 100 18.2 -> 15.3 / 15.3 / 15.7 / 16.4, 20 M x
// 200 42.2 -> 39.1 / 38.3 / 38.5 / 38.8; not bound, 8 M x 40 87 -> 85 / 84 / 79 / 72, 3 M x 100 47.7 -> 47.6 / 46.4 / 45.6 / 45.1.  Below about 1 M rows there is
// nothing to gain (400 k x 2000 7.6 -> 8.3 with four steps).
constexpr int ORDER_ITEMS = 512;
inline int order_shift(int64_t n_rows, bool bound) { return !bound ? 6 : n_rows > 6000000 ? 5 : 3; }

// Nodes of a round looked at by a wavefront, 64 at a time (what is asked about a node behind the last one is 0).
struct WaveNodes {
    int lane;
    template <class F>
    __device__ __forceinline__ int sum(int n, F f) const {
        int c = 0;
        for (int j = 0; j < n; j += 64) c += f(j + lane);
        return wave_sum(c);
    }
    __device__ __forceinline__ int last_start(const int* starts, int n, int at) const { return find_start(starts, n, at); }
    // The node that holds number `at` of the nodes' shares in a row: its share's start, and the number inside the share; false: there are not as many.
    template <class F>
    __device__ __forceinline__ bool find(int n, F share, int& at, int& node, int& from) const {
        for (int j0 = 0; j0 < n; j0 += 64) {
            int f;
            const int k = share(j0 + lane, f), incl = wave_prefix(k), all = __builtin_amdgcn_readlane(incl, 63);
            if (at < all) {
                const int l = __popcll(__ballot(incl <= at));
                at -= __builtin_amdgcn_readlane(incl, l) - __builtin_amdgcn_readlane(k, l);
                node = j0 + l;
                from = __builtin_amdgcn_readlane(f, l);
                return true;
            }
            at -= all;
        }
        return false;
    }
};

template <class Nodes>
struct PartOrder {
    Nodes nodes;
    const int* s_start;
    int n_batch, n_items, shift;
    bool spread;
    int origin, part, first, next;  // first segment of the XCD; the part that holds the last segment asked for: its first one, the next part's

    __host__ __device__ __forceinline__ int segments(int j) const { return j < n_batch ? (j + 1 < n_batch ? s_start[j + 1] : n_items) - s_start[j] : 0; }
    // segments of all nodes in front of part q
    __host__ __device__ __forceinline__ int in_front(int q) const {
        return nodes.sum(n_batch, [&](int j) { return (segments(j) * q) >> shift; });
    }
    __host__ __device__ __forceinline__ void start(const Nodes& w, const int* starts, int count, int items, int block, int sh) {
        nodes = w; s_start = starts; n_batch = count; n_items = items; shift = sh;
        spread = shift > 0 && n_items >= ORDER_ITEMS;
        if (!spread) return;
        part = (block & 7) << (shift - 3);
        first = in_front(part); next = in_front(part + 1);
        origin = first;
    }
    // Segment number `at` of the launch (ascending from call to call): its node and its number among all segments; false: no more
    __host__ __device__ __forceinline__ bool at(int at, int& node, int& item) {
        if (!spread) {
            if (at >= n_items) return false;
            item = at;
            node = nodes.last_start(s_start, n_batch, at);
            return true;
        }
        const int end = ((at & 7) + 1) << (shift - 3);
        const int want = origin + (at >> 3);
        while (want >= next) {
            if (++part == end) return false;
            first = next; next = in_front(part + 1);
        }
        int rest = want - first, from = 0;  // segments of this part in front of it
        if (!nodes.find(n_batch, [&](int j, int& f) { const int n = segments(j); f = (n * part) >> shift; return ((n * (part + 1)) >> shift) - f; }, rest, node, from))
            return false;
        item = s_start[node] + from + rest;
        return true;
    }
};

// The children of an expanded node: `nl` of its rows go left.
__device__ __forceinline__ void put_children(Node* nodes, const BatchEntry& be, int child, int nl, int64_t lg, int64_t lh, int64_t rg, int64_t rh,
                                             int lslot, int rslot) {
    auto put = [&](int which, int64_t begin, int count, int64_t g, int64_t h, int sl) {
        Node* c = &nodes[child + which];
        c->begin = begin; c->count = count; c->sum_g = g; c->sum_h = h; c->n_left = 0; c->buf = be.child_buf; c->slot = sl;
        c->state = 0; c->expanded = 0; c->child = -1; c->leaf_id = -1;
        c->best.gain = 0.0; c->best.feature = -1; c->best.bin = -1;
        c->best.left_g = c->best.left_h = c->best.right_g = c->best.right_h = c->best.left_count = 0;
    };
    put(0, be.begin, nl, lg, lh, lslot);
    put(1, be.begin + nl, be.count - nl, rg, rh, rslot);
}

// The rows of a quarter of segment `item` (256 * R rows, of node nd) to the children's lists, by one wavefront that needs nothing of the
// others.  MODE 1: and the packed gradients; MODE 2 also leaves the rows' destinations in `dpos` (LDS).
template <int MODE, int R, int SUPER>
__device__ __forceinline__ void scatter_wave(const RowSource& rows, int16_t* const* gh_out, const IdxSet& idxs, const BatchEntry& nd, int item, int wave, int lane,
                                             const unsigned long long* __restrict__ masks, const int32_t* __restrict__ seg_counts,
                                             const int32_t* __restrict__ super_counts, int* dpos) {
    constexpr int PART_SEG = 256 * R;
    const int seg = item - nd.seg_start, sup = seg / SUPER;
    const int sbegin = seg * PART_SEG, n = min(nd.count - sbegin, PART_SEG);
    const int n_sup = (nd.n_seg + SUPER - 1) / SUPER;
    const int cbuf = nd.child_buf;
    const bool identity = nd.buf == BUF_ORIGINAL;  // the root's list: row id = position, never stored
    const int32_t* src = idxs.p[nd.buf] + nd.begin + sbegin;
    int32_t* dst = idxs.p[cbuf] + nd.begin;
    const int16_t* gsrc = MODE >= 1 ? rows.gh[nd.buf] + nd.begin + sbegin : nullptr;
    int16_t* gdst = MODE >= 1 ? gh_out[cbuf] + nd.begin : nullptr;
    // everything that is read, in flight together
    int32_t v[R];
    int g16[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int r = min((wave * R + u) * 64 + lane, n - 1);
        v[u] = identity ? (int32_t)(nd.begin + sbegin + r) : src[r];
        g16[u] = MODE >= 1 ? gsrc[r] : 0;
    }
    if (MODE == 0 && identity && rows.code.on()) {  // the root's children are the first lists: entries with their gradients
#pragma unroll
        for (int u = 0; u < R; ++u) v[u] = (int32_t)rows.code.entry((uint32_t)v[u], rows.gh[BUF_ORIGINAL][v[u]]);
    }
    const unsigned long long mk = lane < PART_SEG / 64 ? masks[(int64_t)item * (PART_SEG / 64) + lane] : 0ull;
    int before = SUPER > 1 && lane < seg - sup * SUPER ? seg_counts[item - (seg - sup * SUPER) + lane] : 0;
    int total = 0;
    for (int k = lane; k < n_sup; k += 64) {
        const int c = super_counts[nd.super_start + k];
        total += c;
        before += k < sup ? c : 0;
    }
    static_assert(SUPER <= 64 && PART_SEG / 64 <= 64, "one lane each");
    before = wave_sum(before);  // left rows in earlier segments
    total = wave_sum(total);    // left rows of the node
    const int pc = __popcll(mk);
    const int pre = wave_prefix(pc) - pc;  // left rows of the segment in front of a mask's 64 rows
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int w = wave * R + u, r = w * 64 + lane;
        const uint32_t mlo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mk, w);
        const uint32_t mhi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mk >> 32), w);
        const int left = __builtin_amdgcn_readlane(pre, w) + (int)__builtin_amdgcn_mbcnt_hi(mhi, __builtin_amdgcn_mbcnt_lo(mlo, 0u));
        const bool fl = ((lane < 32 ? mlo : mhi) >> (lane & 31)) & 1u;
        const int dp = fl ? before + left : total + (sbegin - before) + (r - left);
        if (r < n) {
            dst[dp] = v[u];
            if (MODE >= 1) gdst[dp] = (int16_t)g16[u];
            if (MODE == 2) dpos[r] = dp;
        }
    }
}

// What moves the rows of a round beside the split search, where the histogram launch has counted them (CountSource).
struct RowMover {
    RowSource rows;
    IdxSet idxs;
    StepState* step;
    Node* nodes;
    const BatchEntry* batch;
    const int32_t* batch_seg;
    const unsigned long long* masks;
    const int32_t* seg_counts;
    int32_t scan_blocks;  // workgroups in front, which search
};

// Workgroup `block` of `n_blocks` that move the rows; the first one makes the children's records instead, from the left counts.
template <int R>
__device__ void move_rows(const RowMover& mv, int block, int n_blocks) {
    __shared__ int s_start[TABLE_MAX];
    const int n_batch = mv.step->n_batch, n_items = mv.step->n_part_items;
    if (mv.step->done || n_batch <= 0) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    load_batch(mv.batch_seg, n_batch, s_start);
    if (block == 0) {
        __shared__ int s_left[TABLE_MAX];
        for (int t = threadIdx.x; t < n_batch; t += blockDim.x) s_left[t] = 0;
        __syncthreads();
        for (int k = threadIdx.x; k < n_items; k += blockDim.x) {
            int lo = 0, hi = n_batch - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s_start[mid] <= k) lo = mid; else hi = mid - 1;
            }
            atomicAdd(&s_left[lo], mv.seg_counts[k]);
        }
        __syncthreads();
        int built = 0;
        for (int t = threadIdx.x; t < n_batch; t += blockDim.x) {
            const BatchEntry be = mv.batch[t];
            Node* P = &mv.nodes[be.node];
            const int slot = P->slot, child = P->child, nl = s_left[t];
            P->n_left = nl;
            built += be.built_left ? nl : be.count - nl;
            put_children(mv.nodes, be, child, nl, P->best.left_g, P->best.left_h, P->best.right_g, P->best.right_h,
                         be.built_left ? be.new_slot : slot, be.built_left ? slot : be.new_slot);
        }
        built = wave_sum(built);
        if (lane == 0 && built > 0) atomicAdd(&mv.step->prof.rows[mv.rows.code.on() ? HistProfile::CODED : HistProfile::IDS], (unsigned long long)built);
        if (threadIdx.x == 0) mv.step->prof.add(HistProfile::IDS, 0, n_batch);
        return;
    }
    for (int w = (block - 1) * waves + wave; w < 4 * n_items; w += (n_blocks - 1) * waves) {
        const int item = w >> 2;
        const BatchEntry nd = mv.batch[find_start(s_start, n_batch, item)];
        scatter_wave<0, R, 1>(mv.rows, nullptr, mv.idxs, nd, item, w & 3, lane, mv.masks, mv.seg_counts, mv.seg_counts, nullptr);
    }
}

}  // namespace qgbdt
