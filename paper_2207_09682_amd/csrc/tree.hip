// Leaf-wise growth of one tree (greedy splitting of Sec. 3, best-first order of
// Sec. 7), driven from the device.
//
// Best-first growth is sequential by definition: split the open leaf with the
// largest gain, look at its children, repeat.  Its result, however, only depends on
// the gains, so it can be reproduced exactly from a tree that was expanded in a
// different order.  The tree is therefore grown in rounds.  Each round
//   1. replays the best-first order over what is known (commit phase): the open leaf
//      with the largest gain is committed as the next split if it has already been
//      expanded, and its children become open leaves; the replay stops at the first
//      leaf that has not been expanded;
//   2. expands that leaf and, speculatively, other nodes with large gains -- open leaves
//      and, up to three levels ahead, descendants of open leaves that are already expanded -- as
//      far as the leaf budget can still reach them: one batched partition, one batched
//      histogram build for one child of each, one batched subtraction and split
//      search for all children.  Up to a few million rows the build counts the left rows
//      on its way and the search's launch moves the rows (COUNTING_ROWS).
// A speculative expansion that the replay never reaches is simply not part of the
// tree: its node stays a leaf and its row slice is untouched, because children are
// always written to another buffer (buffers rotate with the depth, so a node's rows
// survive the expansions of the levels below it that may run ahead).  Split numbers and leaf ids are
// assigned at commit time, so the result equals the sequential one bit for bit.
//
// The host enqueues whole rounds without reading anything back, as many as the last
// tree took, and behind them the passes over the finished leaves, which return at once
// if the tree is not finished; a word in pinned memory tells it whether more rounds are needed.
#include <algorithm>
#include <chrono>

#include "partition_device.h"
#include "refit_device.h"

namespace qgbdt {

// Row lists: up to this many rows times tiles of features the histogram launch counts the left rows itself (CountSource) and the rows are moved
// beside the split search, which leaves a round four dependent launches (three where no reduce kernel is launched) of six.  Every tile of a
// row group goes through the parents' rows for itself, and a workgroup counts and accumulates one after the other: beyond the line
// the count and scatter kernels, which fill the chip, are the faster way.  A tree of few leaves has few rounds of little work per launch, so its line lies
// higher; one whose rounds have more nodes than there are row-group lanes has lanes with two items, which 64-bit words, accumulated at half the rate, make worse; with more
// than six tiles there are few lanes, and not bound every tile gathers lines of the matrix for its count.  Trees, time without counting over time with it, mean (and
// least) of 1722 shapes drawn from 12 to 1500 features, 15 to 400 bins, 2 to 8 bits, 15 to 511 leaves, by millions of rows x tiles (single shapes vary by 2 %):
//                                                          up to 0.5   0.9         1.4         1.8         2.4         3.0         4.5
//   up to six tiles, leaves <= lanes / 4                   1.15 (1.04) 1.12 (1.06) 1.09 (1.00) 1.08 (1.01) 1.04 (0.98) 1.02 (0.94) 0.99 (0.90)
//                    more leaves                           1.16 (1.06) 1.13 (1.02) 1.08 (0.94) 1.05 (0.92) 1.00 (0.88) 0.98 (0.90) 0.96 (0.85)
//                    64-bit words, leaves > 2 lanes        1.12 (1.09)             1.03 (0.98) 0.99 (0.94) 0.94 (0.86) 0.93 (0.88) 0.91 (0.79)
//   more tiles, bound                                      1.10 (1.04) 1.07 (0.99) 1.04 (0.96) 1.01 (0.91) 0.94 (0.86) 0.94 (0.84) 0.90 (0.78)
//               not bound                                  1.10 (1.05) 1.04 (0.99) 1.00 (0.88) 0.95 (0.80) 0.91 (0.74) 0.85 (0.65)
// Beyond six times the lanes not at all: 57 k x 1323 (11 tiles, 16 lanes), 275 leaves 1426 / 1471 us; 43 k x 640 (5, 48), 277 leaves 983 / 859.
// Single ones, us without / with: 28 features (255 leaves) 1 M 549 / 521, 2 M 690 / 668, not bound 1 M 615 / 541, 2 M 769 / 761, 3 M 863 / 1039; 200 features 500 k 854 /
// 812, 750 k 940 / 965; 136 features, 8-bit hessians 200 k 752 / 690, not bound 600 k 858 / 931; 552 features, 31 bins (31 leaves) 111 k 368 / 327, 333 k 397 / 449.
// 64-bit words of many features in one or two tiles have a line at 0.9 besides, where N x F is above 100 M and the leaves are not few: 0.97 on average beyond it (0.93 to 1.03;
// below it 467 k x 240 1.21, in six tiles 206 k x 1440 1.07).  All 1722 shapes take 5.5 % less time by this rule than without counting (the better of both ways everywhere:
// 5.8 %); 22 of them more than 2 % more.
constexpr int COUNTING_NODES = 6;
static int64_t counting_rows(const HistPlan& plan, bool bound, int num_leaves, int64_t n_bins) {
    const int lanes = count_lanes(plan);
    const bool words64 = plan.acc_width == 32;
    if (num_leaves > COUNTING_NODES * lanes) return 0;
    if (words64 && plan.n_tiles <= 2 && n_bins > 100000000 && 4 * num_leaves > lanes) return 900000;
    if (plan.n_tiles > 6) return bound ? 1600000 : 1100000;
    if (4 * num_leaves <= lanes) return 3000000;
    return words64 && num_leaves > 2 * lanes ? 1400000 : 2000000;
}

// An item of such a launch is one chunk at most (count_item_segs), which for short chunks makes more items than row-group lanes in the rounds of the
// whole matrix: the lanes' second items take as long as the first ones.  Two turns pay up to 2 M rows x tiles, where the second is not nearly
// empty or the items are short and later rounds, whose nodes have fewer rows, outweigh; three never do.  The shapes above of up to six tiles, columns up to 1.4, 1.8, 2.4, 3.0:
//   two turns, the second at least three tenths full, or       1.02 (0.98) 1.04 (0.97) 1.01 (0.91) 0.95 (0.91)
//     more than 32 leaves and items of less than 6144 rows
//   two turns otherwise                                        1.04 (0.98) 0.95 (0.90) 0.93 (0.87) 0.87 (0.78)
//   three and more                                                                     0.95 (0.88) 0.97 (0.91)
static bool counting_turns_pay(const HistPlan& plan, int64_t n_rows, int seg_rows, int num_leaves) {
    const int64_t segs = (n_rows + seg_rows - 1) / seg_rows, turn = (int64_t)count_lanes(plan) * (plan.single_rows / seg_rows);
    if (segs <= turn) return true;
    return segs <= 2 * turn && n_rows * plan.n_tiles <= 2000000 && (10 * segs >= 13 * turn || (num_leaves > 32 && plan.single_rows < 6144));
}

bool counts_rows(const qgbdt_ctx* ctx, const HistPlan& plan, const RowSource& rows, bool bound, int num_leaves) {
    const int64_t N = ctx->shape.n_rows;
    return N * plan.n_tiles <= counting_rows(plan, bound, num_leaves, N * ctx->shape.n_features) && counting_build_ok(ctx, plan, rows) && counting_turns_pay(plan, N, ctx->seg_rows, num_leaves);
}

struct TreeOut {
    qgbdt_tree t;
    int32_t max_leaves;
};

// The answer to the host's request `seq` (0: none).
__device__ __forceinline__ void report_to_host(TreeReport* r, uint64_t seq, bool done, int rounds, int n_expanded, int n_commits, int n_nodes) {
    if (seq == 0) return;
    r->rounds = rounds; r->n_expanded = n_expanded; r->n_commits = n_commits; r->n_nodes = n_nodes;
    __hip_atomic_store(&r->answer, seq * 2 + (done ? 1 : 0), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ void clear_split(qgbdt_split& s) {
    s.gain = 0.0; s.feature = -1; s.bin = -1;
    s.left_g = s.left_h = s.right_g = s.right_h = s.left_count = 0;
}

__device__ __forceinline__ int hist_groups(int64_t count, const HistPlan& plan) {
    const int64_t t = hist_target_rows(plan, count, 1);
    int64_t g = (count + t - 1) / t;
    if (g < 1) g = 1;
    return (int)g;
}

__global__ __launch_bounds__(256) void tree_init_kernel(int64_t N, int F, StepState* step, Node* nodes,
                                                        const int64_t* qtotals_part, int n_part, int root_buf, HistEntry* hist_entries,
                                                        int32_t* hist_counts, ScanPair* pairs,
                                                        int64_t* hist0, int64_t hist_words, HistPlan plan) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = t; i < hist_words; i += stride) hist0[i] = 0;  // (the root's row list is the identity: never stored)
    if (blockIdx.x != 0) return;
    int64_t total[3];  // (a launch of its own for them took 3 us of every tree)
    sum_totals(qtotals_part, n_part, total);
    if (t == 0) {
        step->done = 0; step->n_known = 0; step->n_list = 0; step->n_nodes = 1; step->n_leaves = 1; step->n_commits = 0; step->n_expanded = 0;
        step->n_slots = 1; step->n_batch = 0; step->rounds = 0; step->n_part_items = 0; step->n_scan_items = 1;
        step->hist_units = N * (int64_t)F;
        Node r;
        r.begin = 0; r.count = N; r.sum_g = total[0]; r.sum_h = total[1]; r.n_left = 0; r.buf = root_buf; r.slot = 0;
        r.state = 1; r.expanded = 0; r.child = -1; r.leaf_id = 0;
        clear_split(r.best);
        nodes[0] = r;
        HistEntry e;
        e.begin = 0; e.count = N; e.buf = root_buf; e.slot = 0; e.item_start = 0; e.groups = hist_groups(N, plan);
        hist_entries[0] = e;
        hist_counts[0] = 1; hist_counts[1] = e.groups; hist_counts[2] = e.groups > plan.search_sums ? 1 : 0; hist_counts[3] = (int32_t)N;
        ScanPair sp;
        sp.slot_a = 0; sp.slot_b = -1; sp.parent = -1; sp.a_item = 0; sp.item_start = 0;
        sp.groups = e.groups <= plan.search_sums ? e.groups : 0;
        sp.merged = N > (int64_t)e.groups * plan.single_rows ? 1 : 0; sp.seg_start = 0;
        sp.stat[0].n_rows = N; sp.stat[0].sum_g = r.sum_g; sp.stat[0].sum_h = r.sum_h;
        sp.stat[1] = sp.stat[0];
        pairs[0] = sp;
    }
}

// Barrier for data exchanged through LDS only: unlike __syncthreads it does not wait for the acknowledgement of
// global stores that nobody in the workgroup reads.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ unsigned long long lane_bits(unsigned long long w, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)w, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(w >> 32), lane);
    return ((unsigned long long)hi << 32) | lo;
}

constexpr uint32_t NO_NODE = 0xffffu;
constexpr uint32_t FAR_AHEAD = 0x8000u;  // of a candidate's bottleneck: the node is two or more levels below the open leaf
constexpr uint32_t NODE_ID = 0xfffu;     // of a node's `ids`; the row buffer is in the four bits above
static_assert(6 * MAX_TREE_LEAVES + 1 < 4096 && BUF_ORIGINAL < 16, "a node's id and buffer share 16 bits");

// LDS of the plan kernel, as byte offsets into its dynamic LDS (offsets, not pointers: the compiler then sees LDS accesses
// everywhere; through a struct of generic pointers they became flat ones, three times as slow).
// p_max: all nodes that can be known.  Arrays by gain rank unless noted.
struct PlanLds {
    int key;      // u64 [p_max] gain bits in the new order
    int okey;     // u64 [p_max + 8] gain bits in the kept order; once merged: `info`, what the selection needs of a rank (the last eight places only move the arrays
                  // behind them on by 64 bytes of LDS banks: 464 k x 90 11.06 -> 10.97 us per launch, 1 M x 28 10.41 -> 10.35)
    int ids;      // u32 [p_max] node | row buffer << 12 | left child << 16
    int oids;     // u32 [p_max] the same in the kept order; once merged: `ckey`, u64 [p_max / 2], order of the splits committed now
    int leaf;     // u16 [p_max] leaf id of an open leaf, else NO_NODE
    int oleaf;    // u16 [p_max] the same in the kept order; once merged: `corder`, place among the splits committed now
    int rank_of;  // u16 [p_max] by node: its rank, NO_NODE: committed before or without a gain
    int par;      // u16 [p_max] rank of the parent, NO_NODE: an open leaf
    int shift;    // i32 [p_max] new keys that come right before an old entry, then places of the new ones; after the merge: open splits by bottleneck
    int nkey;     // u64 [2*batch_max + 4] gain bits of last round's children (0: no split)
    int commit;   // u16 [num_leaves] ranks of the splits committed now, in order
    int chosen;   // u16 [batch_max] ranks of the nodes to expand
    int bytes;
};
__host__ __device__ __forceinline__ PlanLds plan_lds_layout(int max_nodes, int batch_max, int num_leaves) {
    const int p = (max_nodes + 3) & ~3;
    PlanLds l;
    l.key = 0; l.okey = l.key + 8 * p; l.nkey = l.okey + 8 * (p + 8); l.ids = l.nkey + 16 * batch_max + 32; l.oids = l.ids + 4 * p;
    l.shift = l.oids + 4 * p; l.leaf = l.shift + 4 * p; l.oleaf = l.leaf + 2 * p; l.rank_of = l.oleaf + 2 * p;
    l.par = l.rank_of + 2 * p; l.commit = l.par + 2 * p; l.chosen = l.commit + ((2 * num_leaves + 7) & ~7);
    l.bytes = l.chosen + ((2 * batch_max + 7) & ~7);
    return l;
}

// The rank whose order key is k: the last of its fields.
__device__ __forceinline__ int key_rank(unsigned long long k) {
    const int tz = __ffsll((long long)k) - 1;
    return (int)((k >> (tz / 12 * 12)) & 0xfffull) - 1;
}

// Leaf id of the node at rank p once its parent is committed.  Left children take their parent's id, the right child
// of the k-th committed split of this call is leaf leaves0 + k; the chain ends at the latest at the node that was an open
// leaf before the call.
__device__ __forceinline__ int leaf_id_at(const uint16_t* leaf, const uint16_t* par, const unsigned long long* info,
                                          const uint16_t* corder, int leaves0, int p) {
    for (;;) {
        const int lf = leaf[p];
        if (lf != (int)NO_NODE) return lf;
        const int q = par[p];
        if ((int)((uint32_t)info[q] & 0xffffu) != p) return leaves0 + corder[q];
        p = q;
    }
}

// Commit phase and choice of the round's batch.  One workgroup of 1024 threads, bound by the latency of its chain of
// phases (about 0.1 us for a barrier, 0.06 us for a dependent LDS access), so everything that is a set of nodes is a
// bit mask over gain ranks (64 ranks to a word, at most 64 words) or a pass with one thread per rank.
//  0. (at most 256 candidates per histogram) The candidates of the histograms scanned last -- one per tile of features --
//     are reduced to their nodes' best splits, by groups of lanes just wide enough that one pass serves all of them, which saves the launch that
//     would do it.
//  1. The known nodes that are not committed and have a gain are kept sorted by it in global memory; last round's
//     children (node ids n_known ..) are merged in: a new one's place is what a search among the old ones finds and a count of the
//     larger new ones.
//  2. Best-first selection (commit the open leaf with the largest gain, its children become open leaves; stop at the
//     first that has not been expanded) without a replay: with distinct gains a node is selected when the *worst* rank
//     on its path from an open leaf is reached, then the worst rank behind that one, and so on -- the order of
//     selection is the lexicographic order of the running maxima of the ranks, read from the node upwards.  Paths are
//     at most five nodes long (nodes are expanded up to three levels below the open leaves), so the order key is one
//     64-bit word of five ranks; the splits committed are the expanded nodes whose key is below that of every node that is not
//     expanded.  Equal gains are resolved by leaf ids, which depend on the order itself: if two known nodes tie, one
//     wavefront replays the selection split by split (a bit per open leaf at its rank, the first set bit is next;
//     0.25 us per split).
//  3. The outputs of the committed splits are written beside the batch's records, at the end: both wait for their nodes then at
//     the same time.
//  4. The batch is chosen with popcounts over the masks: the leaf the selection stopped at, the other open leaves that are
//     not expanded (class 0), then nodes up to n_bufs - 2 levels below expanded open leaves (class 1; a node's rows outlive the
//     expansions of that many levels below it), by rank, if the selection can reach them with the splits that remain: a node
//     comes after all nodes of a larger bottleneck, the smallest gain on the path from the open leaf to the node.  (Counting
//     the nodes of a larger gain of their own instead puts off the descendants of small gains and takes others in their
//     place: 21 against 15 rounds per tree on 200 k x 136.)
//     One level ahead instead of three costs the data that peel a few rows off a large node at every split many rounds:
//     rounds per tree 51 -> 27 (lambdarank 20 M x 200), 27 -> 15 (200 k x 136), 13 -> 11 (10.5 M x 28), 12 -> 10 (464 k x 90).
// Measured per launch against the version that kept all nodes in the order and replayed every split: 20.6 -> 10.1 us
// (1 M x 28, 255 leaves, 20 splits and 44 new nodes per round), 25.6 -> 11.9 us (10.5 M x 28), 24.4 -> 15.6 us
// (20 M x 200, 511 leaves).  With the first candidates requested together with the state, keys merged by search, order keys computed once and
// the outputs last: 11.3 -> 10.5 us (1 M x 28), 11.8 -> 10.9 (464 k x 90), 16.2 -> 13.6 (20 M x 200).
__global__ __launch_bounds__(1024) void tree_plan_kernel(StepState* step, Node* nodes, BatchEntry* batch, int32_t* batch_seg,
                                                         int32_t* super_counts, PlanEntry* list, int32_t* hist_counts, int F, int n_cand, int num_leaves,
                                                         int batch_max, int max_expand, int seg_rows, int seg_supers, int n_bufs, TreeReport* report, uint64_t report_seq, TreeOut out,
                                                         const FeatCand* __restrict__ cand,
                                                         const ScanPair* __restrict__ scan_pairs) {
    // the fields of the growth state this kernel needs and (for the first 1024 ranks) the kept order, in loads that are
    // in flight together
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int max_nodes = 2 * max_expand + 1;
    const int4* sp = reinterpret_cast<const int4*>(step);
    const int4 st0 = sp[0], st1 = sp[1], st2 = sp[2];
    PlanEntry mine = list[min(tid, max_nodes - 1)];
    // Histogram j's candidates are reduced by a group of lanes that holds them all in four loads each; those of the first 32 are
    // requested before it is known how many there are (all of them: more than a compute unit reads in the time that this saves).
    int lg = 0;
    while (lg < 6 && (4 << lg) < n_cand) ++lg;
    const int sl = tid & ((1 << lg) - 1), first_item = tid >> lg;
    const bool ahead = cand != nullptr && first_item < min(32, 2 * batch_max);
    FeatCand fc[4];
    ScanTotals totals;
    if (ahead) {
        load_candidates(cand + (int64_t)first_item * n_cand, n_cand, sl, 1 << lg, fc);
        totals = load_totals(&scan_pairs[first_item >> 1], first_item & 1);
    }
    if (st0.x) {  // done
        if (tid == 0) report_to_host(report, report_seq, true, st1.w, st1.x, st0.w, st0.y);
        return;
    }
    extern __shared__ __attribute__((aligned(16))) unsigned char plan_lds[];
    const PlanLds lay = plan_lds_layout(max_nodes, batch_max, num_leaves);
    unsigned long long* const key = reinterpret_cast<unsigned long long*>(plan_lds + lay.key);
    unsigned long long* const okey = reinterpret_cast<unsigned long long*>(plan_lds + lay.okey);
    unsigned long long* const nkey = reinterpret_cast<unsigned long long*>(plan_lds + lay.nkey);
    uint32_t* const ids = reinterpret_cast<uint32_t*>(plan_lds + lay.ids);
    uint32_t* const oids = reinterpret_cast<uint32_t*>(plan_lds + lay.oids);
    int* const shift = reinterpret_cast<int*>(plan_lds + lay.shift);
    uint16_t* const leaf = reinterpret_cast<uint16_t*>(plan_lds + lay.leaf);
    uint16_t* const oleaf = reinterpret_cast<uint16_t*>(plan_lds + lay.oleaf);
    uint16_t* const rank_of = reinterpret_cast<uint16_t*>(plan_lds + lay.rank_of);
    uint16_t* const par = reinterpret_cast<uint16_t*>(plan_lds + lay.par);
    uint16_t* const commit = reinterpret_cast<uint16_t*>(plan_lds + lay.commit);
    uint16_t* const chosen = reinterpret_cast<uint16_t*>(plan_lds + lay.chosen);
    __shared__ unsigned long long s_open[64], s_exp[64], s_comm[64];
    __shared__ unsigned long long s_c0[64], s_c1[64];  // batch candidates of class 0 and 1
    __shared__ int s_reach[64];                        // open splits by bottleneck, per 64 ranks
    __shared__ int s_nc, s_nnew, s_tie, s_stop, s_nsup;
    __shared__ unsigned long long s_wsum[16];
    __shared__ unsigned long long s_first[8];  // (eight partial results: an atomic on one address is expanded into a loop over the lanes)
    const int n_nodes = st0.y, leaves0 = st0.z, commits0 = st0.w;
    const int n_expanded0 = st1.x, n_slots = st1.y;
    const int n_known = st2.z, n_list = st2.w, n_scan = st2.y;
    const int m_new = n_nodes - n_known;
    const int new_buf = nodes[n_known + min(1023 - tid, m_new - 1)].buf;  // (used when the new nodes are ranked)

    for (int i = tid; i < n_nodes; i += 1024) { rank_of[i] = (uint16_t)NO_NODE; par[i] = (uint16_t)NO_NODE; shift[i] = 0; }
    for (int p = tid; p < n_list; p += 1024) {
        if (p >= 1024) mine = list[p];
        okey[p] = mine.key; oids[p] = mine.ids; oleaf[p] = (uint16_t)mine.leaf;
    }
    if (tid < 64) { s_open[tid] = 0ull; s_exp[tid] = 0ull; s_comm[tid] = 0ull; s_reach[tid] = 0; }
    if (tid == 0) { s_nc = 0; s_nnew = 0; s_tie = 0; s_stop = -1; }
    if (tid < 8) s_first[tid] = ~0ull;
    if (tid < 4) nkey[m_new + tid] = 0ull;
    // Scanned histogram j belongs to node n_known + j: the best splits of last round's children.
    if (cand != nullptr) {
        for (int item = first_item; item < n_scan; item += 1024 >> lg) {
            if (item != first_item || !ahead) {
                load_candidates(cand + (int64_t)item * n_cand, n_cand, sl, 1 << lg, fc);
                totals = load_totals(&scan_pairs[item >> 1], item & 1);
            }
            double gain = 0.0;
            int feature = -1;
            reduce_candidates(fc, cand + (int64_t)item * n_cand, n_cand, totals, &nodes[n_known + item].best, sl, 1 << lg, gain, feature);
            if (sl == 0)
                nkey[item] = (feature >= 0 && gain > 0.0) ? (unsigned long long)__double_as_longlong(gain) : 0ull;
        }
    } else {
        for (int t = tid; t < m_new; t += 1024) {
            const qgbdt_split* b = &nodes[n_known + t].best;
            const double gain = b->gain;
            nkey[t] = (b->feature >= 0 && gain > 0.0) ? (unsigned long long)__double_as_longlong(gain) : 0ull;
        }
    }
    lds_barrier();
    // merge: old entries keep their order and come first among equal keys; new ones follow by node id.  A new key's place among the
    // old ones is searched for and counted there; the running sum of these counts is what the old ones move by.
    // (Counting the larger keys for every entry instead is a matter of LDS bandwidth: 128 new and 200 old ones 2.1 us, 170 and 300 4.5 us.)
    for (int t0 = 0; t0 < m_new; t0 += 64) {  // among the new keys: a wavefront's share comes in runs of 4, the entries behind the end are 0
        const int t = t0 + lane;
        const unsigned long long kb = t < m_new ? nkey[t] : 0ull;
        if (kb == 0ull) continue;  // (per lane: a child without a split has no rank)
        int c = 0;
        for (int u0 = 4 * wave; u0 < m_new; u0 += 64) {
#pragma unroll
            for (int u = 0; u < 4; ++u) c += (nkey[u0 + u] > kb || (nkey[u0 + u] == kb && u0 + u < t)) ? 1 : 0;
        }
        if (c) atomicAdd(&shift[n_list + t], c);
    }
    const int half = n_list > 0 ? 1 << (31 - __clz(n_list)) : 0;
    for (int t0 = 1024 - 64 * (wave + 1); t0 < m_new; t0 += 1024) {  // among the old ones (by the last wavefronts)
        const int t = t0 + lane;
        const unsigned long long kb = t < m_new ? nkey[t] : 0ull;
        const int found = __popcll(__ballot(kb != 0ull));
        if (lane == 0 && found) atomicAdd(&s_nnew, found);
        if (kb == 0ull) continue;
        int at = 0;
        for (int d = half; d > 0; d >>= 1)
            if (at + d <= n_list && okey[at + d - 1] >= kb) at += d;
        if (at < n_list) { atomicAdd(&shift[at], 1); atomicAdd(&s_reach[at >> 6], 1); }
        if (at) atomicAdd(&shift[n_list + t], at);
    }
    lds_barrier();
    const int moved = wave_prefix(s_reach[lane]) - s_reach[lane];  // new keys in front of every 64 old ones
    const int P = n_list + s_nnew;  // ranks in use
    for (int p0 = wave * 64; p0 < n_list; p0 += 1024) {
        const int p = p0 + lane;
        const int by = __builtin_amdgcn_readlane(moved, p0 >> 6) + wave_prefix(p < n_list ? shift[p] : 0);
        if (p >= n_list) continue;
        const uint32_t id = oids[p];
        const int q = p + by;
        key[q] = okey[p]; ids[q] = id; leaf[q] = oleaf[p];
        rank_of[id & NODE_ID] = (uint16_t)q;
    }
    for (int t = 1023 - tid; t < m_new; t += 1024) {  // (from the last thread down: other wavefronts than the loop above, mostly)
        const unsigned long long kb = nkey[t];
        if (kb == 0ull) continue;
        const int q = shift[n_list + t];
        const int buf = t < 1024 ? new_buf : nodes[n_known + t].buf;
        key[q] = kb; ids[q] = (uint32_t)(n_known + t) | ((uint32_t)buf << 12) | (NO_NODE << 16);
        leaf[q] = (uint16_t)(n_known + t == 0 ? 0u : NO_NODE);  // the root is an open leaf from the start
        rank_of[n_known + t] = (uint16_t)q;
    }
    lds_barrier();
    if (tid < 64) s_reach[tid] = 0;
    // of every rank: the ranks of both children (info), expanded, tie with the next rank; of the children: their parent
    unsigned long long* const info = okey;
    uint16_t* const corder = oleaf;
    for (int p = tid; p < P; p += 1024) {
        const uint32_t child = ids[p] >> 16;
        uint32_t lo = 0xffffffffu;
        if (child != NO_NODE) {
            const uint32_t rl = rank_of[child], rr = rank_of[child + 1];
            lo = rl | (rr << 16);
            if (rl != NO_NODE) par[rl] = (uint16_t)p;
            if (rr != NO_NODE) par[rr] = (uint16_t)p;
        }
        const uint32_t tie = (p + 1 < P && key[p + 1] == key[p]) ? 2u : 0u;
        info[p] = ((unsigned long long)(tie | (child != NO_NODE ? 1u : 0u)) << 32) | lo;
        corder[p] = (uint16_t)NO_NODE; shift[p] = 0;
        if (tie) s_tie = 1;
    }
    lds_barrier();
    const int budget = num_leaves - 1 - commits0;
    unsigned long long* ckey = reinterpret_cast<unsigned long long*>(oids);
    if (!s_tie) {
        // order key of rank p: running maxima of (rank + 1) on the path up to the open leaf, the largest first, 12 bits
        // each; a path has at most n_bufs nodes
        static_assert(ROW_BUFS <= 5 && 6 * MAX_TREE_LEAVES + 1 < 4096, "fields of the order key");
        auto order_key = [&](int p) {
            unsigned long long k = (unsigned long long)(p + 1) << 48;
            int top = p;
            for (int q = par[p]; q != (int)NO_NODE; q = par[q])
                if (q > top) { k = (k >> 12) | ((unsigned long long)(q + 1) << 48); top = q; }
            return k;
        };
        unsigned long long mine_key = 0ull;  // of the thread's first rank
        for (int p = tid; p < P; p += 1024) {
            const unsigned long long k = order_key(p);
            if (p < 1024) mine_key = k;
            if (!((info[p] >> 32) & 1ull)) atomicMin(&s_first[lane & 7], k);
        }
        lds_barrier();
        unsigned long long first = s_first[0];
#pragma unroll
        for (int u = 1; u < 8; ++u) first = min(first, s_first[u]);
        for (int p = tid; p < P; p += 1024) {
            if (!((info[p] >> 32) & 1ull)) continue;
            const unsigned long long k = p < 1024 ? mine_key : order_key(p);
            if (k < first) ckey[atomicAdd(&s_nc, 1)] = k;
        }
        lds_barrier();
        const int nc = s_nc;
        for (int c = tid; c < nc; c += 1024) {
            const unsigned long long k = ckey[c];
            int o = 0;
            for (int u = 0; u < nc; ++u) o += ckey[u] < k ? 1 : 0;
            const int p = key_rank(k);
            if (o < budget) { commit[o] = (uint16_t)p; corder[p] = (uint16_t)o; }
        }
    } else {
        for (int p0 = wave * 64; p0 < P; p0 += 1024) {
            const int p = p0 + lane;
            const unsigned long long mo = __ballot(p < P && leaf[p] != NO_NODE);
            if (lane == 0) s_open[p0 >> 6] = mo;
        }
        lds_barrier();
        if (wave == 0) {
            unsigned long long ow = s_open[lane];  // this lane's word of open leaves
            int nc = 0, stop = 0;
            bool out_of_leaves = false;
            for (;;) {
                const unsigned long long any = __ballot(ow != 0ull);
                if (any == 0ull || nc >= budget) { out_of_leaves = true; break; }
                const int src = __ffsll((long long)any) - 1;
                int r = src * 64 + __ffsll((long long)lane_bits(ow, src)) - 1;
                if ((info[r] >> 33) & 1ull) {  // equal gains: the lowest leaf id of the run's open leaves
                    int best = r, bl = leaf_id_at(leaf, par, info, corder, leaves0, r);
                    for (int q = r; (info[q] >> 33) & 1ull;) {
                        ++q;
                        if (!((lane_bits(ow, q >> 6) >> (q & 63)) & 1ull)) continue;
                        const int ql = leaf_id_at(leaf, par, info, corder, leaves0, q);
                        if (ql < bl) { bl = ql; best = q; }
                    }
                    r = __builtin_amdgcn_readfirstlane(best);
                }
                const unsigned long long inf = info[r];
                if (!((inf >> 32) & 1ull)) { stop = r; break; }  // the next split is not known yet
                const int rl = (int)((uint32_t)inf & 0xffffu), rr = (int)((uint32_t)inf >> 16);
                if (lane == (r >> 6)) ow &= ~(1ull << (r & 63));
                if (lane == (rl >> 6)) ow |= 1ull << (rl & 63);  // (NO_NODE >> 6 is no lane)
                if (lane == (rr >> 6)) ow |= 1ull << (rr & 63);
                if (lane == 0) { commit[nc] = (uint16_t)r; corder[r] = (uint16_t)nc; }
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                nc += 1;
            }
            if (lane == 0) { s_nc = nc; s_stop = stop; s_first[0] = out_of_leaves ? ~0ull : 0ull; }
        }
    }
    __syncthreads();  // (also: the best splits stored above are read below)
    const int n_commit = min(s_nc, budget);
    unsigned long long first_open = s_first[0];
#pragma unroll
    for (int u = 1; u < 8; ++u) first_open = min(first_open, s_first[u]);
    const bool done = n_commit >= budget || first_open == ~0ull;  // (no leaf with a gain is left)
    // the leaf the selection stopped at (an order key ends with the node's own rank)
    const int stop = s_tie ? s_stop : key_rank(first_open);
    // the masks after the commits
    for (int p0 = wave * 64; p0 < P; p0 += 1024) {
        const int p = p0 + lane;
        bool open = false, expanded = false, committed = false;
        if (p < P) {
            expanded = (info[p] >> 32) & 1ull;
            committed = corder[p] != NO_NODE;
            int worst = p, level = 0;  // the largest rank on the path to the open leaf, the levels on it
            if (!committed) {
                for (int q = par[p]; q != (int)NO_NODE && corder[q] == NO_NODE; q = par[q]) { ++level; worst = max(worst, q); }
                atomicAdd(&shift[worst], 1);
                atomicAdd(&s_reach[worst >> 6], 1);
            }
            open = !committed && level == 0;
            const bool ahead = level > 0 && level <= n_bufs - 2 && !expanded;
            reinterpret_cast<uint32_t*>(info)[2 * p + 1] = !ahead ? NO_NODE : (uint32_t)worst | (level > 1 ? FAR_AHEAD : 0u);  // (the flags are not read again)
        }
        const unsigned long long mo = __ballot(open), me = __ballot(expanded), mc = __ballot(committed);
        if (lane == 0) { s_open[p0 >> 6] = mo; s_exp[p0 >> 6] = me; s_comm[p0 >> 6] = mc; }
    }
    // Outputs and node states of the splits committed above: behind the choice of the batch, which does not wait for the nodes then, and
    // by the last threads, beside the batch's records.
    auto put_commits = [&]() {
        unsigned long long units = 0ull;
        for (int c = 1023 - tid; c < n_commit; c += 1024) {
            const int r = commit[c], lid = leaf_id_at(leaf, par, info, corder, leaves0, r), k = commits0 + c;
            const int i = (int)(ids[r] & NODE_ID), ch = (int)(ids[r] >> 16);
            const Node nd = nodes[i];
            out.t.split_leaf[k] = lid; out.t.split_feature[k] = nd.best.feature; out.t.split_bin[k] = nd.best.bin;
            out.t.split_gain[k] = nd.best.gain;
            out.t.split_stats[4 * k + 0] = nd.best.left_g; out.t.split_stats[4 * k + 1] = nd.best.left_h;
            out.t.split_stats[4 * k + 2] = nd.best.right_g; out.t.split_stats[4 * k + 3] = nd.best.right_h;
            out.t.split_n_left[k] = nd.n_left;
            const int64_t nl = nd.n_left, nr = nd.count - nd.n_left;
            units += (unsigned long long)((nl <= nr ? nl : nr) * (int64_t)F);
            // a child that has itself been committed in this call is internal; its own iteration says so
            const int q0 = rank_of[ch], q1 = rank_of[ch + 1];
            if (q0 == (int)NO_NODE || corder[q0] == NO_NODE) { nodes[ch].state = 1; nodes[ch].leaf_id = lid; }
            if (q1 == (int)NO_NODE || corder[q1] == NO_NODE) { nodes[ch + 1].state = 1; nodes[ch + 1].leaf_id = leaves0 + c; }
            nodes[i].state = 2;
        }
        if (1023 - 64 * wave - 63 < n_commit) {  // (the wavefront has splits)
            for (int o = 32; o > 0; o >>= 1) units += __shfl_xor(units, o);
        }
        if (lane == 0 && units) atomicAdd(reinterpret_cast<unsigned long long*>(&step->hist_units), units);
        if (tid == 0) { step->n_commits = commits0 + n_commit; step->n_leaves = leaves0 + n_commit; step->n_known = n_nodes; }
    };
    lds_barrier();
    if (done) {
        put_commits();
        if (tid == 0) {
            step->done = 1; step->n_batch = 0; step->n_part_items = 0; step->n_scan_items = 0;
            hist_counts[0] = 0; hist_counts[1] = 0; hist_counts[2] = 0;
            report_to_host(report, report_seq, true, st1.w, n_expanded0, commits0 + n_commit, n_nodes);
        }
        return;
    }
    if (tid == 0) report_to_host(report, report_seq, false, st1.w, n_expanded0, commits0 + n_commit, n_nodes);
    // One expansion is certain (the leaf the selection stopped at); expansions beyond those
    // that the remaining certain ones will need may be spent on speculation.  That leaf is always in the batch, so the
    // next call commits at least one split and `spare` stays >= 0: never more than max_expand nodes are expanded, which
    // the tables of nodes and histograms are made for.
    const int remaining = budget - n_commit;
    const int spare = (max_expand - n_expanded0) - remaining;
    int want = 1 + (spare > 0 ? spare : 0);
    if (want > remaining) want = remaining;
    if (want > batch_max) want = batch_max;
    // The last rank that the selection can reach as a bottleneck: fewer than `remaining` open splits have a better one.  Every
    // wavefront finds it for itself, first the word of 64 ranks, then the rank.
    // Nodes two or more levels ahead are guesses on guesses: while many splits remain they have to be within half of them.
    // Rounds / expansions / time per tree with half and with all: 10.5 M x 28 11 / 285 / 1885 us and 10 / 324 / 1911 us,
    // 20 M x 200 27 / 620 / 10.91 ms and 23 / 761 / 11.01 ms; the last 32 splits without that limit: 200 k x 136 699 -> 669 us.
    const int in_front = wave_prefix(s_reach[lane]) - s_reach[lane];
    auto last_reached = [&](int splits) {
        auto last_below = [&](int n) { return 63 - __clzll((long long)__ballot(n < splits)); };  // (lane 0's always is)
        const int w = last_below(in_front);
        const int d = 64 * w + lane < P ? shift[64 * w + lane] : 0;
        return 64 * w + last_below(__builtin_amdgcn_readlane(in_front, w) + wave_prefix(d) - d);
    };
    const int reach = last_reached(remaining), reach_far = last_reached(max(remaining / 2, min(remaining, 32)));
    for (int p0 = wave * 64; p0 < P; p0 += 1024) {
        const int p = p0 + lane, w = p0 >> 6;
        const unsigned long long near = __ballot(p <= reach || p == stop);
        const uint32_t worst = p < P ? (uint32_t)(info[p] >> 32) : NO_NODE;
        const unsigned long long c1 = __ballot(worst != NO_NODE && (int)(worst & ~FAR_AHEAD) <= (worst & FAR_AHEAD ? reach_far : reach));
        if (lane == 0) { s_c0[w] = s_open[w] & ~s_exp[w] & near; s_c1[w] = c1; }
    }
    lds_barrier();
    // candidates of both classes (class 1 in the upper half) and committed splits in front of every word
    const bool in = lane < ((P + 63) >> 6);
    const int c01 = in ? __popcll(s_c0[lane]) | (__popcll(s_c1[lane]) << 16) : 0, cc = in ? __popcll(s_comm[lane]) : 0;
    const int n_cls = wave_prefix(c01) - c01, n_comm = wave_prefix(cc) - cc;
    const int n_all = __builtin_amdgcn_readlane(n_cls + c01, 63);
    const int n0 = n_all & 0xffff, n_batch = min(n0 + (n_all >> 16), want);
    for (int p0 = wave * 64; p0 < P; p0 += 1024) {
        const int p = p0 + lane, w = p0 >> 6;
        const int pre = __builtin_amdgcn_readlane(n_cls, w), gone = __builtin_amdgcn_readlane(n_comm, w);
        if (p >= P) continue;
        const unsigned long long bit = 1ull << lane, below = bit - 1ull;
        const unsigned long long cw = s_comm[w], c0 = s_c0[w], c1 = s_c1[w];
        uint32_t id = ids[p];
        if ((c0 | c1) & bit) {  // order of the batch: the leaf the selection stopped at, class 0 by gain, class 1 by gain
            int o = (c0 & bit) ? (pre & 0xffff) + __popcll(c0 & below) : n0 + (pre >> 16) + __popcll(c1 & below);
            if (c0 & bit) o = p == stop ? 0 : p < stop ? o + 1 : o;  // (leaves of equal gain may be in front of it by rank)
            if (o < n_batch) {
                chosen[o] = (uint16_t)p;
                id = (id & 0xffffu) | ((uint32_t)(n_nodes + 2 * o) << 16);
            }
        }
        if (!(cw & bit)) {
            PlanEntry e;
            e.key = key[p]; e.ids = id; e.leaf = (s_open[w] & bit) ? (uint32_t)leaf_id_at(leaf, par, info, corder, leaves0, p) : NO_NODE;
            list[p - gone - __popcll(cw & below)] = e;
        }
    }
    lds_barrier();
    put_commits();
    // the batch's records: segments of the batched partition, new histogram slots, child ids
    BatchEntry be;
    be.n_seg = 0;
    if (tid < n_batch) {
        const int p = chosen[tid], i = (int)(ids[p] & NODE_ID);
        const Node* nd = &nodes[i];
        be.begin = nd->begin; be.count = (int32_t)nd->count; be.node = i; be.buf = nd->buf;
        be.feature = nd->best.feature; be.bin = nd->best.bin;
        be.n_seg = (int)(((uint32_t)be.count + (uint32_t)seg_rows - 1u) / (uint32_t)seg_rows);
        be.new_slot = n_slots + tid;
        // the children's rows go to the first buffer that neither holds the node's own nor those of a node above it that
        // may yet stay a leaf (at most n_bufs - 1 in all); with two in turn most of the time, rather than all in turn,
        // the lists stay in the caches (2 M x 40 of 16-bit bins 1 %)
        uint32_t taken = 1u << be.buf;
        for (int q = par[p]; q != (int)NO_NODE && corder[q] == NO_NODE; q = par[q]) taken |= 1u << ((ids[q] >> 12) & 15u);
        be.child_buf = __ffs((int)~taken) - 1;
        // (counting build) the child that is built from its rows: the one of fewer rows as far as the hessians tell
        be.built_left = nd->best.left_h <= nd->best.right_h ? 1 : 0;
        be.pad = 0;
        nodes[i].expanded = 1;
        nodes[i].child = n_nodes + 2 * tid;
    }
    // (segments and groups of segments in one scan: groups in the upper half, at most 2^31 / 512 segments below)
    unsigned long long incl = (unsigned long long)be.n_seg | ((unsigned long long)((be.n_seg + PART_SUPER - 1) / PART_SUPER) << 32);
    const unsigned long long own = incl;
    for (int o = 1; o < 64 && o < n_batch; o <<= 1) { const unsigned long long u = __shfl_up(incl, o); if (lane >= o) incl += u; }
    if (n_batch > 64) {  // uniform over the workgroup
        if (lane == 63) s_wsum[wave] = incl;
        lds_barrier();
        for (int k = 0; k < wave; ++k) incl += s_wsum[k];
    }
    if (tid < n_batch) {
        be.seg_start = (int)(uint32_t)(incl - own);
        be.super_start = seg_supers ? (int)((incl - own) >> 32) : be.seg_start;
        batch[tid] = be;
        batch_seg[tid] = be.seg_start;
    }
    if (seg_supers) {
        if (tid == n_batch - 1) s_nsup = (int)(incl >> 32);
        lds_barrier();
        for (int t = tid; t < s_nsup; t += 1024) super_counts[t] = 0;  // the count kernel adds to them
    }
    if (tid == n_batch - 1) {
        step->n_part_items = (int)(uint32_t)incl;
        step->n_batch = n_batch;
        step->n_nodes = n_nodes + 2 * n_batch;
        step->n_slots = n_slots + n_batch;
        step->n_expanded = n_expanded0 + n_batch;
        step->rounds = st1.w + 1;
        step->n_scan_items = 2 * n_batch;
        step->n_list = P - n_commit;
    }
}

__global__ __launch_bounds__(1024) void tree_finalize_kernel(const StepState* step, const Node* nodes,
                                                             const float* delta, int parts, int extra, RefitUnit* units,
                                                             int2* leaves, TreeOut out) {
    __shared__ LeafLayout s;
    if (step->done == 0) return;  // (uniform) the host enqueues this pass before it knows
    const int n = step->n_leaves;
    const double dg = (double)delta[0], dh = (double)delta[1];
    for (int l = threadIdx.x; l < out.max_leaves; l += blockDim.x) {
        if (l >= n) {
            out.t.leaf_begin[l] = 0; out.t.leaf_count[l] = 0; out.t.leaf_sum_g[l] = 0; out.t.leaf_sum_h[l] = 0;
            out.t.leaf_value_quant[l] = 0.0;
        }
    }
    for (int i = threadIdx.x; i < step->n_nodes; i += blockDim.x) {
        const Node S = nodes[i];
        if (S.state != 1) continue;
        const int l = S.leaf_id;
        out.t.leaf_begin[l] = S.begin; out.t.leaf_count[l] = S.count;
        out.t.leaf_sum_g[l] = S.sum_g; out.t.leaf_sum_h[l] = S.sum_h;
        out.t.leaf_value_quant[l] = (S.sum_h > 0 && dh > 0.0) ? -((double)S.sum_g * dg) / ((double)S.sum_h * dh) : 0.0;
        s.begin[l] = S.begin; s.count[l] = S.count; s.buf[l] = S.buf;
    }
    if (threadIdx.x == 0) {
        *out.t.n_leaves = n;
        out.t.delta[0] = delta[0]; out.t.delta[1] = delta[1];
        *out.t.hist_units = step->hist_units;
    }
    __syncthreads();
    layout_leaves(s, n, out.max_leaves, parts, extra, units, leaves);
}

// LDS of the plan kernel for this context's node capacity.
static size_t plan_kernel_lds(const qgbdt_ctx* ctx, int num_leaves) {
    return (size_t)plan_lds_layout(ctx->max_nodes, ctx->batch_max, num_leaves).bytes;
}

int prepare_tree_kernels(qgbdt_ctx* ctx) {
    const size_t plan_lds = plan_kernel_lds(ctx, ctx->shape.max_leaves);
    if (ctx->max_nodes > 4096 || plan_lds + 8192 > 160 * 1024)  // (masks and static words come on top)
        return set_error(ctx, QGBDT_E_UNSUPPORTED, "max_leaves=%d needs %zu bytes of LDS for the growth bookkeeping (limit 160 KB)",
                         ctx->shape.max_leaves, plan_lds);
    if (plan_lds > 48 * 1024)
        QG_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(tree_plan_kernel),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)plan_lds));
    return QGBDT_OK;
}

// Waits for the answer to request `seq` or a later one in pinned memory: the stream's work behind it goes on meanwhile.  (Copying the status word
// and waiting for the stream left the GPU idle for 15 to 25 us at the end of every tree.)  The stream is asked now and then whether it is still at work, so that an error ends the wait.
static int wait_for_report(qgbdt_ctx* ctx, uint64_t seq, bool* done) {
    const auto answered = [&]() {
        const uint64_t a = __atomic_load_n(&ctx->report->answer, __ATOMIC_ACQUIRE);
        *done = a & 1;
        return a >> 1 >= seq;
    };
    for (auto next = std::chrono::steady_clock::now() + std::chrono::milliseconds(1);;) {
        for (int k = 0; k < 64; ++k) {
            if (answered()) return QGBDT_OK;
            __builtin_ia32_pause();
        }
        if (std::chrono::steady_clock::now() < next) continue;
        const hipError_t e = hipStreamQuery(ctx->stream);
        if (e == hipSuccess) {
            if (answered()) return QGBDT_OK;
            return set_error(ctx, QGBDT_E_HIP, "the plan kernel left no answer");
        }
        if (e != hipErrorNotReady) return set_error(ctx, QGBDT_E_HIP, "hipStreamQuery failed: %s", hipGetErrorString(e));
        next = std::chrono::steady_clock::now() + std::chrono::milliseconds(1);
    }
}

int run_grow_tree(qgbdt_ctx* ctx, const uint8_t* bins, const float* g, const float* h, const qgbdt_params* p,
                  uint32_t iteration, const qgbdt_tree* tout, int32_t* row_idx_out) {
    const int64_t N = ctx->shape.n_rows;
    const int F = ctx->shape.n_features, nb = ctx->shape.n_bins;
    const int64_t W = (int64_t)F * nb;
    TreeOut out;
    out.t = *tout;
    out.max_leaves = ctx->shape.max_leaves;

    // 32|32 words of the total histograms must hold the root's sums
    const bool check_totals = N > max_rows_for_width(p->bits_g, p->bits_h, 32);
    int rc = launch_quantize(ctx, g, h, N, p->bits_g, p->bits_h, p->seed, iteration, p->rounding, ctx->gh,
                             ctx->delta, check_totals ? ctx->qtotals : nullptr, ctx->ghf);
    if (rc != QGBDT_OK) return rc;
    if (check_totals) {
        int64_t tot[3];
        QG_HIP(ctx, hipMemcpyAsync(tot, ctx->qtotals, sizeof(tot), hipMemcpyDeviceToHost, ctx->stream));
        QG_HIP(ctx, hipStreamSynchronize(ctx->stream));
        if (tot[1] > 0xffffffffLL || tot[2] > 0x7fffffffLL)
            return set_error(ctx, QGBDT_E_OVERFLOW_RISK,
                             "quantized totals (sum h~ = %lld, sum |g~| = %lld) do not fit 32|32 packed bins",
                             (long long)tot[1], (long long)tot[2]);
    }
    // most frequent bins of the bound matrix: left out by the wide-row histogram kernels, rebuilt by the split search
    const bool skip_ok = ctx->mfb_features > 0 && ctx->bins_t && ctx->bound_bins == (const void*)bins;
    // (the large tiles that skipping makes worthwhile pay for contiguous rows only: the gathered builds of the
    // rounds keep the ordinary tiles -- 20M x 200: 212 against 197 us per launch)
    const HistPlan plan = make_hist_plan(ctx->shape, p->bits_g, p->bits_h, p->acc_width, false);
    const HistPlan root_plan = make_hist_plan_for(ctx->shape, p->bits_g, p->bits_h, p->acc_width, N, skip_ok,
                                                  ((uintptr_t)bins & 15) == 0);  // the root's build alone: contiguous rows
    const uint16_t* mfb = skip_ok ? ctx->mfb : nullptr;
    // Row sources: buffer BUF_ORIGINAL = the caller's matrix and the quantized gradients in original order;
    // the others are what the partition writes (see RowSource).
    RowSource rows;
    IdxSet idxs;
    // the feature-major copy serves only the matrix it was made from
    const uint8_t* bins_t = (ctx->bins_t && ctx->bound_bins == (const void*)bins) ? ctx->bins_t : nullptr;
    ctx->seg_supers = part_supers(N, bins_t != nullptr) ? 1 : 0;
    // Without the feature-major copy the partition's count gathers a line of the row-major matrix per row, once per level; keeping
    // the rows in leaf order reads and writes the whole row at every level instead.  Rows of 36 bytes and more are cheaper to
    // gather (20 M x 48 5.99 / 7.45 ms per tree, index / ordered), shorter ones too while the matrix is in the caches, those of up to 20 bytes less long the more
    // levels a tree has.  The line lies where both were level before the counting pass took the order of the XCDs and histogram launches counted; since then
    // index trees are the faster ones on both sides of it, up to 10 to 30 M rows.  Time ordered / index now with 31, 127 and 511 leaves: 1 M x 16 1.44 1.33 1.31, 1.5 M 1.31
    // 1.23 1.27, 2 M 1.29 1.19 1.17, 3 M 1.17 1.14 1.16, 7 M 1.28 1.20 1.12; 1 M x 20 1.23 1.24 1.28, 2 M 1.18 1.09 1.04, 3 M 1.17 1.12 1.10, 7 M 1.26 1.16 1.07; 2 M x 24 1.21 1.12 1.09, 4.5 M 1.32 1.25
    // 1.17 (4 M, 5 bits 1.35 1.30 1.28), 7 M 1.24 1.17 1.07; 1 M x 28 1.28 1.22 1.20, 4.5 M 1.33 1.26 1.16, 7 M 1.28 1.19 1.12; 7 M x 32 1.29 1.24 1.20; with 31 and 255 leaves 10 M x 16 1.21 1.06,
    // 16 M 1.04 0.97, 30 M 0.98 0.86; 10 M x 20 1.15 1.02, 30 M 0.93 0.84; 10 M x 28 1.20 1.09, 30 M 1.01 0.94; 10 M x 32 1.23 1.18, 30 M 1.08 1.02.  (With the
    // feature-major copy moving row ids wins throughout: 10.5 M x 28 1.64 against 2.54 ms.)
    // Without ordered rows the packed gradients still move with the row ids (2 bytes per moved row): a gathered
    // build then reads them in sequence, which takes one of the ~2.2 cache lines per sparse narrow row away.
    // A matrix that the caches hold gathers cheaply anyway and gains nothing from the move (1 M x 28: 1.15 to
    // 1.21 against 1.16 ms per tree).
    // Where the row id and the quantized gradients fit 32 bits together the list's entries hold both (RowCode) and neither
    // is gathered nor moved apart.
    int layout = p->row_layout;
    int levels = 4;
    while (F <= 20 && (1 << levels) < p->num_leaves) ++levels;
    if (layout == QGBDT_ROWS_AUTO)
        layout = (ctx->ordered != 0 && !bins_t && N * F * (36 - F) * levels > (int64_t)4000 << 20) ? QGBDT_ROWS_ORDERED
                 : ((int64_t)N * F * ctx->shape.bin_bytes >= (int64_t)128 << 20) ? QGBDT_ROWS_IDS_GH : QGBDT_ROWS_IDS;
    const bool ordered = layout == QGBDT_ROWS_ORDERED;
    rows.code = PLAIN_ROWS;
    int id_bits = 1;
    while (((int64_t)1 << id_bits) < N) ++id_bits;
    if (p->row_layout == QGBDT_ROWS_AUTO && !ordered && id_bits + p->bits_g + p->bits_h <= 32) {
        rows.code = {(uint32_t)(((uint64_t)1 << id_bits) - 1), id_bits, p->bits_h, 32 - p->bits_g, p->bits_h == 0 ? 1 : 0};
        layout = QGBDT_ROWS_IDS;
    }
    const bool gh_lists = layout != QGBDT_ROWS_IDS;
    if (ordered && !ctx->ordered)
        return set_error(ctx, QGBDT_E_WORKSPACE, "the workspace has no room for leaf-ordered copies of the rows");
    ctx->tree_layout = rows.code.on() ? QGBDT_ROWS_IDS_CODED : layout;
    for (int b = 0; b < ROW_BUFS; ++b) {
        rows.bins[b] = ordered && b < COPY_BUFS ? ctx->obins[b] : bins;
        rows.gh[b] = gh_lists ? ctx->ogh[b] : ctx->gh;
        idxs.p[b] = ctx->idx[b];
    }
    rows.gh_pos = (gh_lists && !ordered) ? 1 : 0;
    rows.pitch = F * ctx->shape.bin_bytes;
    rows.bins[BUF_ORIGINAL] = bins; rows.gh[BUF_ORIGINAL] = ctx->gh; idxs.p[BUF_ORIGINAL] = ctx->idx[0];
    // the root's rows are the original arrays under the identity list
    const int root_buf = BUF_ORIGINAL;

    // the copy at a pitch of whole cache lines serves the matrix it was made from, like the feature-major one
    RowSource hist_rows = rows;
    if (bins_t && ctx->bins_p && plan.wide_v == 8 && !ordered) {
        for (int b = 0; b <= ROW_BUFS; ++b) hist_rows.bins[b] = ctx->bins_p;
        hist_rows.pitch = padded_pitch(ctx->shape);
    }

    // up to 256 candidates per histogram the plan kernel reduces them itself (one launch less per round)
    const int n_cand = scan_candidates(ctx->shape);
    const FeatCand* fused_cand = n_cand <= 256 ? ctx->cand : nullptr;
    int blocks = (int)((W + 255) / 256);
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(tree_init_kernel, dim3(blocks), dim3(256), 0, ctx->stream, N, F, ctx->step,
                       ctx->nodes, ctx->qtotals_part, quantize_parts(g, h, ctx->gh, N), root_buf, ctx->hist_entries, ctx->hist_counts, ctx->scan_pairs,
                       ctx->hist_pool, W, root_plan);
    ctx->next_hist_is_root = 1;
    rc = launch_hist(ctx, root_plan, rows, idxs, false, ((uintptr_t)bins & 15) == 0,
                     ctx->hist_entries, ctx->hist_counts, ctx->hist_pool,
                     (N + hist_target_rows(root_plan, N, 1) - 1) / hist_target_rows(root_plan, N, 1),  // the build's row groups
                     mfb, root_plan.search_sums);
    if (rc != QGBDT_OK) return rc;
    const bool counting = !ordered && !gh_lists && counts_rows(ctx, plan, hist_rows, bins_t != nullptr, p->num_leaves);
    ctx->tree_counting = counting ? 1 : 0;
    auto search_splits = [&](const HistPlan& hp, int max_pairs, const RowMover* mover) {
        int rc = launch_scan_pairs(ctx, ctx->hist_pool, ctx->scan_pairs, &ctx->step->n_scan_items, max_pairs, ctx->delta,
                                   p->min_data_in_leaf, p->min_sum_hessian, ctx->cand, mfb, &hp, mover);
        if (rc != QGBDT_OK || fused_cand) return rc;
        return launch_reduce_items(ctx, ctx->cand, ctx->scan_pairs, &ctx->step->n_scan_items, 2 * max_pairs,
                                   &ctx->nodes->best, sizeof(Node), ctx->step);
    };
    rc = search_splits(root_plan, 1, nullptr);
    if (rc != QGBDT_OK) return rc;

    const size_t plan_lds = plan_kernel_lds(ctx, p->num_leaves);  // at most what prepare_tree_kernels allowed
    const int round_cap = 4 * ctx->shape.max_leaves + 8;  // every round commits or expands at least one node
    auto plan_batch = [&](uint64_t report_seq) {
        hipLaunchKernelGGL(tree_plan_kernel, dim3(1), dim3(1024), plan_lds, ctx->stream, ctx->step, ctx->nodes, ctx->batch,
                           ctx->batch_seg, ctx->super_counts, ctx->plan_list, ctx->hist_counts, F, n_cand, p->num_leaves,
                           ctx->batch_max, ctx->max_expand, ctx->seg_rows, ctx->seg_supers, ordered ? COPY_BUFS : ROW_BUFS, ctx->report,
                           report_seq, out, fused_cand, ctx->scan_pairs);
    };
    auto expand_batch = [&]() {  // partition, histograms and split search of the nodes the plan kernel has chosen
        if (counting) {
            const CountSource count = {bins_t, N, ctx->step, ctx->nodes, ctx->batch, ctx->batch_seg, ctx->part_masks, ctx->seg_counts,
                                       ctx->hist_entries, ctx->hist_counts, ctx->scan_pairs, ctx->seg_rows, ctx->batch_max};
            int rc = launch_hist(ctx, plan, hist_rows, idxs, true, false, ctx->hist_entries, ctx->hist_counts, ctx->hist_pool,
                                 plan.max_lanes, mfb, plan.search_sums, &count);
            if (rc != QGBDT_OK) return rc;
            const RowMover mover = {rows, idxs, ctx->step, ctx->nodes, ctx->batch, ctx->batch_seg, ctx->part_masks, ctx->seg_counts, 0};
            return search_splits(plan, ctx->batch_max, &mover);
        }
        int rc = launch_batch_partition_count(ctx, rows, bins_t, ordered);
        if (rc != QGBDT_OK) return rc;
        rc = launch_batch_partition_scatter(ctx, rows, ordered, plan);
        if (rc != QGBDT_OK) return rc;
        rc = launch_hist(ctx, plan, hist_rows, idxs, !ordered, ordered, ctx->hist_entries,
                         ctx->hist_counts, ctx->hist_pool, plan.max_lanes, mfb, plan.search_sums);
        if (rc != QGBDT_OK) return rc;
        return search_splits(plan, ctx->batch_max, nullptr);
    };
    auto leaf_passes = [&]() {  // what is left to do when the tree is finished; returns at once while it is not
        ctx->tree_passes += 1;
        hipLaunchKernelGGL(tree_finalize_kernel, dim3(1), dim3(1024), 0, ctx->stream, ctx->step, ctx->nodes, ctx->delta,
                           refit_parts(N), refit_extra(N), ctx->refit_units, ctx->refit_leaves, out);
        QG_HIP(ctx, hipGetLastError());
        return launch_gather_refit(ctx, idxs, rows.code.id_mask, row_idx_out, out.t.n_leaves, out.t.leaf_value);
    };
    ctx->tree_rounds = 0;
    ctx->tree_passes = 0;
    for (; ctx->tree_rounds < ctx->rounds_hint; ++ctx->tree_rounds) {
        plan_batch(0);
        rc = expand_batch();
        if (rc != QGBDT_OK) return rc;
    }
    // One more plan commits what the last round made known and tells whether the tree is finished; behind it, what is left to do
    // if it is.  A tree that needs a round or two more than the last one gets each after the answer to the one before.
    bool done = false;
    for (int missing = 0;; ++missing) {
        plan_batch(++ctx->report_seq);
        rc = leaf_passes();
        if (rc != QGBDT_OK) return rc;
        rc = wait_for_report(ctx, ctx->report_seq, &done);
        if (rc != QGBDT_OK) return rc;
        if (done || missing == 2) break;
        rc = expand_batch();  // (the plan has chosen a batch already)
        if (rc != QGBDT_OK) return rc;
        ctx->tree_rounds += 1;
    }
    if (!done) {
        // From the third missing round on a round is enqueued before the host has read the answer of the one in front of it, so that
        // the GPU does not wait for the host, and the leaf passes at the end; the last round finds the tree finished (9 us).  Each
        // after the answer, with the leaf passes behind it, cost 5 us per missing round.  First tree of a context (10 rounds enqueued up
        // front), each after the answer / one ahead / three per answer: 100 k x 50 with 56 rounds 2216 / 2030 / 2068 us, 20 M x 200 with
        // 21 rounds 10.76 / 10.66 / 10.71 ms; one round missing: 1 M x 28 658 / 673 / 700 us, 464 k x 90 702 / 711 / 742 us.
        auto one_more = [&]() {
            const int rc = expand_batch();
            ctx->tree_rounds += 1;
            plan_batch(++ctx->report_seq);
            return rc;
        };
        rc = one_more();
        while (rc == QGBDT_OK && !done) {
            if (ctx->tree_rounds > round_cap) return set_error(ctx, QGBDT_E_HIP, "tree growth did not finish in %d rounds", ctx->tree_rounds);
            rc = one_more();
            if (rc == QGBDT_OK) rc = wait_for_report(ctx, ctx->report_seq - 1, &done);
        }
        if (rc != QGBDT_OK) return rc;
        rc = leaf_passes();
        if (rc != QGBDT_OK) return rc;
        // (nothing that is still to run writes the report when the call returns)
        rc = wait_for_report(ctx, ctx->report_seq, &done);
        if (rc != QGBDT_OK) return rc;
    }
    ctx->rounds_hint = ctx->report->rounds > 0 ? ctx->report->rounds : 1;
    return QGBDT_OK;
}

}  // namespace qgbdt
