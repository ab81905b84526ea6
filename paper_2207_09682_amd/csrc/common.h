// Internal declarations shared by the HIP translation units of libqgbdt.
// Nothing here is part of the public boundary (see include/qgbdt.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>

#include "../../include/qgbdt.h"

namespace qgbdt {

// ---- device-side bookkeeping of one tree -----------------------------------

// A node of the tree being grown.  Nodes are created in pairs when their parent is
// expanded (partitioned, histograms built, best split searched); a node becomes an
// open leaf when its parent's split is committed in best-first order.
struct Node {
    int64_t begin, count;  // slice of the row list `buf`
    int64_t sum_g, sum_h;  // quantized totals
    int64_t n_left;        // rows sent left by this node's split (valid once expanded)
    int32_t buf;           // which of the row lists holds the slice (RowSource)
    int32_t slot;          // histogram slot in the pool
    int32_t state;         // 0 waiting for its parent's commit, 1 open leaf, 2 internal (split committed)
    int32_t expanded;      // children exist (their rows, histograms and best splits are known)
    int32_t child;         // left child id (right = child + 1), -1 if none
    int32_t leaf_id;       // valid once the node is an open leaf
    qgbdt_split best;      // best split of this node (feature < 0: none)
};

// What the histogram launches have had to do.  Counted by the first thread of each from a total that the tables hold.  (Their makers, which
// counted before, end at once and waited for the three atomics: stand-alone builds 3 M x 28 by row list 26.3 / 25.9 us, 500 k x 13 15.8 / 15.4, a
// tree's first launch 0.3 us.  Walking the table instead held up every launch of many builds.)  Launches that select their rows
// (CountSource) learn the total last: there the kernel behind them counts.
struct HistProfile {
    enum { CONTIGUOUS = 0, IDS = 1, CODED = 2 };  // rows: contiguous, gathered by row id, gathered by entries that hold their gradients (RowCode)
    unsigned long long rows[3];
    unsigned long long launches;  // histogram launches that had rows
    unsigned long long builds;    // histogram builds served by those launches
    __device__ __forceinline__ void add(int kind, int64_t n_rows, int n_builds) {  // (atomics: nothing waits for the old values)
        atomicAdd(&rows[kind], (unsigned long long)n_rows);
        atomicAdd(&launches, 1ull);
        atomicAdd(&builds, (unsigned long long)n_builds);
    }
};

struct ScanPair;

// State of the growth of one tree.
struct StepState {
    int32_t done;        // 1: tree finished, later kernels return at once
    int32_t n_nodes, n_leaves, n_commits, n_expanded, n_slots;
    int32_t n_batch;     // nodes expanded in the current round
    int32_t rounds;
    int32_t n_part_items;  // row segments of the current round's partitions
    int32_t n_scan_items;  // histograms to scan in the current round
    int32_t n_known;       // nodes that have passed through tree_plan_kernel (all but the last round's children)
    int32_t n_list;        // entries of the kept gain order (see tree_plan_kernel)
    int64_t hist_units;    // rows*features of the histogram builds the sequential algorithm performs
    HistProfile prof;
};

// What a plan kernel tells the host when it is asked to, in pinned memory: how far the tree is, and behind it the number of the
// request with the answer to "is it finished" in the lowest bit.
struct TreeReport {
    int32_t rounds, n_expanded, n_commits, n_nodes;
    uint64_t answer;
};

// One node expanded in the current round, with everything the partition kernels need of it (one 56-byte record
// instead of a look-up in the node table that depends on it).
struct BatchEntry {
    int64_t begin;      // the node's rows: slice of buffer `buf`
    int32_t count;
    int32_t node;
    int32_t seg_start;  // first partition segment of this node
    int32_t n_seg;
    int32_t new_slot;   // histogram slot of the child that is built from its rows
    int32_t buf;
    int32_t feature, bin;  // its split
    int32_t super_start;   // first of its groups of PART_SUPER segments (without such counters: of its segments)
    int32_t child_buf;     // buffer its children's rows go to
    int32_t built_left;    // (counting build) 1: the left child's histogram is built from its rows, 0: the right one's
    int32_t pad;
};

// One known node whose split is not committed yet and has a gain, in the gain order kept from round to round.
struct PlanEntry {
    unsigned long long key;  // bits of the gain (> 0): ordered like the gain
    uint32_t ids;            // node id in 12 bits, row list in the next four, left child's id in the upper half (0xffff: not expanded)
    uint32_t leaf;           // leaf id, 0xffff: not an open leaf (its parent's split is not committed)
};

// Best candidate of one (leaf, tile of features) pair produced by the scan kernel.
struct FeatCand {
    double gain;
    int64_t left;  // packed prefix word (G_L | H_L)
    int32_t bin;   // -1: no valid candidate
    int32_t feature;
};

// One histogram build: a row slice accumulated into one slot, cut into `groups` row groups
// that are the work items [item_start, item_start + groups) of the launch.
struct HistEntry {
    int64_t begin, count;
    int32_t buf;   // index buffer (gathered builds)
    int32_t slot;  // histogram slot relative to the base pointer
    int32_t item_start;
    int32_t groups;
};

// Pitch of the copy of a bound matrix that the gathered builds of a tree read 8 bytes at a time (hist_wide_kernel; 0: none): whole cache
// lines.  These builds are bound by the requests of 64 bytes, and the lines behind them, that a CU can have outstanding: a 32-byte piece
// of a row of 200 bytes takes 1.375 requests, the row 2.5 lines instead of 2.  Where that costs at most 30 % more bytes per row (104, 120, 200, 216, 232 and
// 248 features), and the matrix is larger than what the caches hold.  Trees without / with: 20 M x 200 9864 / 9367 us, 8 M x 232 3999 / 3714, 4 M x 200 2280 / 2154,
// 3 M x 120 1277 / 1158, 2 M x 200 1470 / 1414, 1.5 M x 104 (156 MB) 742 / 747.  Contiguous rows gain little: one build of 20 M x 200 1425 / 1390 us.  Matrices read 16 bytes at a
// time have no such copy: 400 k x 2000 loses (at a pitch of 2048 185 / 212 us, gathered 67 / 68), 112 to 240 features would gain in 32-bit words (8 M x 112 2774 / 2414 us, 6 M x 208
// 3297 / 3072, 5 M x 224 2876 / 2742, 5 M x 240 3109 / 2831, 1.5 M x 208 1104 / 1076) and not in 64-bit ones (3 M x 240 2307 / 2306).
inline int padded_pitch(const qgbdt_shape& s) {
    const int F = s.n_features, pitch = (F + 127) / 128 * 128;
    return s.bin_bytes == 1 && F > 64 && F < 256 && F % 16 == 8 && 10 * pitch <= 13 * F && s.n_rows * F >= (int64_t)256 << 20 ? pitch : 0;
}

// Work descriptor of one stand-alone row partition.
struct PartWork {
    int64_t begin, count;
    int32_t feature, bin;
};

struct HistPlan {
    int32_t ft;          // features per workgroup tile (a multiple of 4 unless the tile is the whole row)
    int32_t ftp;         // padded tile width in LDS words
    int32_t dpr;         // dwords per row per tile = ceil(ft/4)
    int32_t rows_per_it; // rows one wavefront covers per iteration
    int32_t n_tiles;     // feature tiles
    int32_t threads;     // workgroup size
    int32_t lds_bytes;
    int32_t chunk_rows;  // rows accumulated between two merges of the local bins
    int32_t max_groups;  // row groups whose workgroups are resident at once
    int32_t max_lanes;   // most workgroups along the row axis of a launch (a multiple of 8)
    int32_t min_rows_per_group;
    int32_t acc_width;   // 16: packed 32-bit words in LDS (g~ sums above hshift, h~ sums below), 32: packed 32|32 words
    int32_t hshift;      // bits of the hessian field of a 32-bit local word: 16, or the split that takes more rows
    int32_t flat_lanes;  // > 0: contiguous slices may use the flat 16-byte-load kernel with this many lanes
    int32_t flat_rows;   // rows per wavefront iteration of that kernel
    int32_t max_items;    // most work items (row groups) of one launch = slots of the partial-histogram buffer
    int32_t slot_bytes;   // bytes of one (item, tile) slot: the tile's local bins, padded to 16 bytes
    int32_t search_sums;  // tree growth: builds of at most this many row groups are added up by the split search (0x7fffffff: all)
    int32_t single_rows;  // a group of at most this many rows is accumulated in one chunk by every kernel variant
    int32_t pad16;        // local bins keep 4 unused words after every 16 features (wide rows, 16-byte loads)
    int32_t wide_v;       // > 0: wide rows are read in pieces of this many bytes per lane (8 or 16)
    int32_t pieces;        // > 0: 16-byte pieces per tile row, of the kernel that reads such pieces
    int32_t turn, contig_turn; // of that kernel: rows by which the order of a piece's bins moves on from one 32 columns of a tile to the next
    int32_t contig_dwords; // 1: contiguous rows are read by dwords all the same
    int32_t ragged;       // feature count not a multiple of 4: unaligned dword loads, last dword of a tile row partial
    int32_t bytewise;     // no dword kernel applies (rows or a tile narrower than 4 bytes): one byte load per bin
    int32_t two_level;    // byte-stream kernel with 32-bit working words folded into 64-bit words in LDS after every chunk
                          // (one large contiguous build: few, long row groups; slots hold the 64-bit words)
};

// Rows per row group when `total` rows of `n_entries` builds are shared out.
//  - As many groups as workgroups are resident at once, and no more: every build ends with a group that is not full, so one
//    place per build but the first is left for them.  (Without it a few workgroups took a second group when the others had
//    ended: 10.5 M x 28 2169 -> 2050 us per tree, 400 k x 2000 1241 -> 1185 us, 2 M x 40 of 16-bit bins 906 -> 888 us.)
//  - Twice as many where the matrix has several tiles of features and a group still has 4096 rows: the last tile is narrower,
//    and what its workgroups leave idle goes to those that start later; below 4096 the bins handed over twice cost more.  Time of
//    a tree against never doubling, with the line at 512 / 4096 / 8192 rows per group: 4 M x 200 -4.5 / -4.7 / 0.0 %, 3 M x 500
//    -2.2 / -2.7 / -3.1 %, 4 M x 136 (8-bit hessians) +4.5 / +0.7 / +0.2 %, 9 M x 40 of 16-bit bins -0.5 / -0.9 / -0.8 %; 20 M x 200
//    -2.8 % with 4096, -2.5 % with 8192, -0.5 % with 16384; with 512 1 M x 200 +11 %, 1 M x 500 +5.6 %, 2 M x 40 +5.5 %, 400 k x 2000 +3.5 %.
//  - Not fewer than min_rows_per_group rows, unless the launch would then have fewer than 64 workgroups: a group of
//    2048 rows takes a wavefront through 16 dependent rounds of loads (100 k x 50 434 -> 385 us per tree with 650 rows; where
//    the chip is busy smaller groups only have more bins to hand over, 1 M x 28 676 -> 690 us with 1024).
//  - When the item table has room, no group is larger than one chunk, so that none merges through atomics.
__host__ __device__ inline int64_t hist_target_rows(const HistPlan& p, int64_t total, int n_entries) {
    int64_t groups = p.max_groups;
    if (p.n_tiles > 1 && total / (2 * groups) >= 4096) groups *= 2;
    const int64_t places = groups - (n_entries - 1);
    groups = places > (groups + 1) / 2 ? places : (groups + 1) / 2;
    int64_t t = (total + groups - 1) / groups;
    const int64_t few = total * p.n_tiles / 64;
    int64_t least = p.min_rows_per_group;
    if (few < least) least = few > 512 ? few : 512;
    if (t < least) t = least;
    if (t > p.single_rows) {
        const int64_t room = (int64_t)p.max_items - n_entries - 1;
        if (total / p.single_rows < room) t = p.single_rows;
        else if (room > 0 && (total + room - 1) / room > t) t = (total + room - 1) / room;
    }
    return t;
}

// In tree growth the split search sums a build's slots itself when there are at most this many (a thread's loads of them are
// all in flight at once); builds of more row groups are summed up by the reduce kernel, which spreads them over the
// whole chip and otherwise returns at once.  Trees with 8 / 64: 400 k x 2000 1283 / 1396 us, 2 M x 40 of 16-bit bins
// 924 / 980 us, 1 M x 28 the same.
// Where no build has more than 33 groups (hist_target_rows, count_item_segs) the search adds them all up and the reduce kernel, 3 us of every round with the gap in
// front of it, is not launched: up to 2^14 rows in one tile, 2^17 rows times tiles in several, unless the bits
// of a forced word width allow short groups only.  Trees of 15 / 63 leaves with the launch, without it: 16 k x 28 194 / 312, 189 / 300 us, 8 k x 500 of 63 bins 205 / 370, 193 /
// 347, 33 k x 500 239 / 404, 229 / 387, 44 k x 90 229 / 341, 222 / 328, 65 k x 100 253 / 398, 254 / 392, 65 k x 56 (8 bits) 228 / 340, 237 / 333, 33 k x 200 249 / 410, 266 /
// 421; beyond the lines 32 k x 50 215 / 347, 220 / 345, 131 k x 100 263 / 393, 278 / 397, 66 k x 200 260 / 395, 276 / 412 (65 k x 500 254 / 369, 241 / 351).  With 8 bits in 32-bit
// words (groups of 129 rows) 16 k x 28 280 / 308 us, 30 k x 100 410 / 518 us, 65 k x 68 339 / 540 us.
constexpr int REDUCE_ABOVE = 8;
constexpr int SEARCH_SUMS_MOST = 33;  // (32 and one that rounding may add)
constexpr int ALL_GROUPS = 0x7fffffff;

// Counting build (CountSource): workgroups of 1024 threads, one per CU, and row-group lanes in multiples of 8.
constexpr int COUNT_THREADS = 1024;
__host__ __device__ inline int count_lanes(const HistPlan& p) { return 256 / p.n_tiles >= 16 ? 256 / p.n_tiles / 8 * 8 : 8; }
// Segments per work item, `total` of them in the round's `n_entries` builds: no more items than workgroups, with a place left for the item
// of every build that is not full (a CU with two of them takes twice as long: 1 M x 28 19 -> 25 us), of at least 1024 rows (512 or 2048
// rows: within 3 % on 10 k to 1 M rows) and of one chunk, so that nothing is merged.  Where the search adds up every build, no build has more than
// SEARCH_SUMS_MOST items (the plan sees to it where the chunk is the limit).  Trees of 15 / 63 leaves without / with that limit: 65 k x 56, 8 bits
// 258 / 235, 354 / 331 us, x 120 256 / 237, 386 / 368; 44 k x 90 230 / 222, 336 / 329; 34 k x 50, 5 bits 235 / 225, 356 / 347.
__host__ __device__ inline int count_item_segs(const HistPlan& p, int total, int n_entries, int seg_rows) {
    const int lanes = count_lanes(p), places = max(lanes - (n_entries - 1), (lanes + 1) / 2);
    int k = max((total + places - 1) / places, (1024 + seg_rows - 1) / seg_rows);
    if (p.search_sums == ALL_GROUPS) k = max(k, (total + SEARCH_SUMS_MOST - 1) / SEARCH_SUMS_MOST);
    return max(min(k, p.single_rows / seg_rows), 1);
}

// Where a gathered build's row groups lie in its list.  A list ascends, so position in the list is position in the matrix, and lines
// that hold rows of several builds (or of a build's neighbouring rows) are fetched once if the builds pass them on one XCD at about
// the same time: the groups that an XCD holds of a build (work items go round-robin to the XCDs) share one stretch of the list, the n-th of
// the XCD number, and take its blocks of rows in turn.  Rows of one or two lines (hist_piece_kernel): per launch against groups of consecutive
// rows 10.5 M x 28 63.7 -> 58.5 us, 2 M x 40 of 16-bit bins 26.9 -> 26.6; rows of many lines share none (20 M x 200 157.6 / 158.8, 400 k x 2000 66.7 / 67.8:
// hist_wide_kernel keeps consecutive rows).
struct GroupPlace {
    int first, n, own;  // groups of the XCDs in front, groups of this XCD, which of them this one is
};
__host__ __device__ __forceinline__ GroupPlace group_place(int item_start, int groups, int item) {
    // every XCD has groups / 8 of them, and those that the last, incomplete turn of eight meets, which starts at the first one's XCD, one more
    const int x = item & 7, s = item_start & 7;
    const uint32_t turn = (1u << (groups & 7)) - 1u, more = ((turn << s) | (turn >> (8 - s))) & 0xffu;
    return {x * (groups >> 3) + (int)__builtin_popcount(more & ((1u << x) - 1u)), (groups >> 3) + (int)((more >> x) & 1u), (item - item_start) >> 3};
}

// One unit of the passes over finished leaves (refit, score update): in every part of the row order, piece
// (part * n + unit - first) of the leaf's rows, piece_rows long.
struct RefitUnit {
    int64_t begin, count;  // the leaf's rows
    int64_t piece_rows;
    int32_t first, n;      // the leaf's units of a part: [first, first + n)
    int32_t leaf;
    int32_t buf;           // index buffer that holds the leaf's rows (tree growth)
};

struct RowMover;

// Where the rows of a slice live: in one of ROW_BUFS buffers, in ordered mode of COPY_BUFS.  The children of a node share its
// slice in another buffer, which holds the rows of no node above them that may yet stay a leaf (tree_plan_kernel).  Buffer
// BUF_ORIGINAL is the caller's data in original row order (bin matrix, quantized gradients), where the root lives.
// In ordered mode (narrow rows) the buffers hold leaf-ordered copies of the bin rows and
// packed gradients.  Otherwise the bin rows are gathered from the original matrix by row id;
// with `gh_pos` set the packed gradients still travel with the row ids (gh[b][p] belongs to
// row idx[b][p]: 2 more bytes per moved row, and a gathered build reads them in sequence
// instead of one more cache line per row), without it they are gathered from gh[BUF_ORIGINAL].
// How many there are decides how far a tree may be grown ahead of its commits (tree_plan_kernel): nodes up to n - 2 levels
// below an open leaf can be expanded while that leaf's rows are still there.  Five row lists cost 12 bytes per row more than
// three; a tree of 20 M x 200 (lambdarank) takes 51 rounds with three lists, 30 with four, 27 with five; six would save one or two
// more (replayed on the host).  The leaf-ordered copies of the rows themselves stay three: five gain 1 % on 2.5 M x 28.
constexpr int ROW_BUFS = 5;
constexpr int COPY_BUFS = 3;
constexpr int BUF_ORIGINAL = ROW_BUFS;
// In index mode an entry of a row list is the row id, or, where both fit 32 bits, the row id with the row's quantized gradients
// above it: h~ from bit id_bits on, g~ in the top bits.  A gathered build then reads one list and the bin rows and nothing else.
// Per launch against gathered gradients: 1 M x 28 12.9 -> 11.6 us, 464 k x 90 15.3 -> 13.9 us; against gradients in lists of their
// own (2 bytes per row that the partition moves as well) 10.5 M x 28: build 66.1 -> 63.5 us, scatter 25.5 -> 15.6 us.
struct RowCode {
    uint32_t id_mask;              // all ones: row ids only
    int32_t id_bits, h_bits;       // h_bits 0: constant hessians, h~ = 1
    int32_t g_shift, h_one;
    __host__ __device__ bool on() const { return id_mask != 0xffffffffu; }
    // (g~ high byte, h~ low byte), sign-extended, as the int16 lists hold it
    __device__ __forceinline__ int gh(uint32_t e) const {
        return ((int32_t)e >> g_shift) * 256 + (int)(__builtin_amdgcn_ubfe(e, (uint32_t)id_bits, (uint32_t)h_bits) | (uint32_t)h_one);
    }
    __device__ __forceinline__ uint32_t entry(uint32_t row, int ghv) const {
        return row | (h_one ? 0u : (uint32_t)(ghv & 0xff) << id_bits) | ((uint32_t)(ghv >> 8) << g_shift);
    }
};
constexpr RowCode PLAIN_ROWS = {0xffffffffu, 32, 0, 0, 0};
struct RowSource {
    const uint8_t* bins[ROW_BUFS + 1];
    const int16_t* gh[ROW_BUFS + 1];
    int32_t gh_pos;
    int32_t pitch;  // bytes from a row to the next; more than a row's own: the padded copy of a bound matrix (padded_pitch)
    RowCode code;
};
// A histogram launch over the rows of a round's nodes that finds out itself which of them go to the child that it builds, and leaves
// the masks and counts of the left rows behind for whoever moves them.  bins_t null: no feature-major copy.
struct CountSource {
    const uint8_t* bins_t;
    int64_t n_rows;
    const StepState* step;
    const Node* nodes;
    const BatchEntry* batch;
    const int32_t* batch_seg;
    unsigned long long* masks;
    int32_t* seg_counts;
    HistEntry* entries;  // tables of the reduce kernel and the search, which it makes on the way
    int32_t* counts;
    ScanPair* pairs;
    int32_t seg_rows, batch_max;
};
constexpr int SELECT_ROWS = 4096;  // rows of a parent that a workgroup goes through at a time
struct RowDest {
    uint8_t* bins[COPY_BUFS];
    int16_t* gh[ROW_BUFS];
};
struct IdxSet {
    int32_t* p[ROW_BUFS + 1];  // (the root's list is the identity and never stored: the last one stands for it)
};

}  // namespace qgbdt

struct qgbdt_ctx {
    qgbdt_shape shape;
    hipStream_t stream;
    int device;
    // the caller's workspace block (qgbdt_set_workspace); every device pointer below points into it
    void* ws_base;
    size_t ws_bytes;
    uint32_t ws_flags;
    // sizes derived from the shape
    int batch_max;   // most nodes expanded per round
    int max_expand;  // most expansions per tree (sequential ones plus speculative ones)
    int max_nodes;
    int seg_rows;   // rows per segment of the batched partition
    int seg_supers; // 1: with counters per PART_SUPER segments (of the tree being grown)
    int max_seg;
    int max_super;
    int rounds_hint;
    int tree_layout;  // QGBDT_ROWS_* that the last tree was grown with
    int tree_counting;  // 1: its histogram launches counted the left rows
    int tree_rounds, tree_passes;  // rounds and passes over its leaves that were enqueued for it
    // workspace
    int ordered;           // the workspace holds leaf-ordered copies of the rows (narrow rows, QGBDT_WS_ROW_COPIES)
    uint8_t* obins[qgbdt::COPY_BUFS];  // [N][F] each (ordered mode), else null
    int16_t* ogh[qgbdt::ROW_BUFS];     // [N] each: packed gradients in the order of idx[b]
    int32_t* idx[qgbdt::ROW_BUFS];     // [N] each
    uint8_t* bins_t;       // [F][N] feature-major copy of the bound bin matrix (QGBDT_WS_BIND, filled by qgbdt_bind_bins), else null
    uint8_t* bins_p;       // [N][padded_pitch] copy of the bound matrix (wide rows; QGBDT_WS_BIND), else null
    uint16_t* mfb;         // [F] most frequent bin of each feature of the bound matrix when it holds most rows, else 0xffff
    int mfb_features;      // features with such a bin (0: no skipping)
    const void* bound_bins; // the matrix that copy was made from
    int16_t* gh;           // [N]
    float2* ghf;           // [N] (g, h) interleaved, written by the quantizer for the refit's gather
    float* gbuf;           // [N] loss derivatives of a boosting iteration run by the library (QGBDT_WS_BOOST), else null
    float* hbuf;           // [N]
    int64_t* hist_pool;    // [max_expand + 1][nb*F]
    void* hist_partials;   // [max_items][n_tiles] local bins of the row groups, summed by the reduce kernel
    size_t hist_partials_bytes;
    uint8_t* flags;        // [N] partition flags (stand-alone partition)
    unsigned long long* part_masks;  // [max_seg][rows per segment / 64] a bit per row of the round's partitions: goes left
    int64_t* part_counts;  // [PART_GROUPS] (stand-alone partition)
    int32_t* seg_counts;   // [max_seg] left rows per partition segment
    int32_t* super_counts; // [max_super] left rows per group of PART_SUPER segments of a node
    float* absmax_part;    // [QUANT_PARTS][2] per-workgroup max|g|, max h
    int64_t* qtotals_part; // [QUANT_PARTS][3] per-workgroup quantized totals
    int64_t* qtotals;      // [3] sum g~, sum h~, sum |g~|
    float* delta;          // [2]
    qgbdt::Node* nodes;          // [max_nodes]
    qgbdt::PlanEntry* plan_list; // [max_nodes] uncommitted nodes by descending gain, kept from round to round
    qgbdt::StepState* step;      // [1]
    qgbdt::BatchEntry* batch;    // [batch_max]
    int32_t* batch_seg;          // [batch_max] their first segments, for the search segment -> node
    qgbdt::FeatCand* cand;       // [2*batch_max][F]
    qgbdt::HistEntry* hist_entries;  // [batch_max]
    int32_t* hist_counts;        // [4] entries, items, 1: an entry has more groups than the split search adds up (HistPlan::search_sums), rows of all entries
    qgbdt::ScanPair* scan_pairs; // [batch_max]
    qgbdt::RefitUnit* refit_units;  // [max_leaves + REFIT_EXTRA] of the leaves last laid out
    int2* refit_leaves;          // [max_leaves + 1] first unit and units of a leaf; behind the leaves: number of units
    double* refit_partial;       // [refit_parts][max_leaves + REFIT_EXTRA][2], a leaf's pieces consecutive
    int64_t* tmp_i64;            // [8]
    qgbdt::TreeReport* report;     // pinned host memory
    uint64_t report_seq;           // requests so far
    // profiling
    int profiling;
    hipEvent_t* ev;
    int ev_cap, ev_used;
    unsigned char* ev_root;  // [ev_cap / 2] 1: the launch was a tree's root build (all rows, contiguous)
    int next_hist_is_root;
    void* static_scratch;  // this device's copy of the library's fixed scratch array (entry points that allocate nothing)
    char err[512];
};

namespace qgbdt {

__device__ __forceinline__ long long readlane64(long long v, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((unsigned long long)v >> 32), lane);
    return (long long)(((unsigned long long)hi << 32) | lo);
}

// Sum over the 64 lanes with DPP moves (no LDS traffic); the result is uniform.
__device__ __forceinline__ int wave_sum(int v) {
#define QG_DPP_ADD(x, ctrl, rmask) ((x) + __builtin_amdgcn_update_dpp(0, (x), ctrl, rmask, 0xf, false))
    v = QG_DPP_ADD(v, 0x111, 0xf);  // row_shr:1
    v = QG_DPP_ADD(v, 0x112, 0xf);  // row_shr:2
    v = QG_DPP_ADD(v, 0x114, 0xf);  // row_shr:4
    v = QG_DPP_ADD(v, 0x118, 0xf);  // row_shr:8: lane 15 of a row holds the row's sum, lane k the sum up to k
    v = QG_DPP_ADD(v, 0x142, 0xa);  // row_bcast:15 into rows 1 and 3
    v = QG_DPP_ADD(v, 0x143, 0xc);  // row_bcast:31 into rows 2 and 3
    return __builtin_amdgcn_readlane(v, 63);
}
// Inclusive prefix sum over the lanes, the same way.
__device__ __forceinline__ int wave_prefix(int v) {
    v = QG_DPP_ADD(v, 0x111, 0xf);
    v = QG_DPP_ADD(v, 0x112, 0xf);
    v = QG_DPP_ADD(v, 0x114, 0xf);
    v = QG_DPP_ADD(v, 0x118, 0xf);
    v = QG_DPP_ADD(v, 0x142, 0xa);
    v = QG_DPP_ADD(v, 0x143, 0xc);
    return v;
#undef QG_DPP_ADD
}

// The last of the n ascending `starts` (in LDS, the first one 0) that is not above `at`, by a whole wavefront: 64 of them are compared
// at a time (a binary search is a chain of LDS accesses of about 0.05 us each).
__device__ __forceinline__ int find_start(const int* starts, int n, int at) {
    int c = 0;
    for (int k = 0; k < n; k += 64) {
        const int i = k + (int)(threadIdx.x & 63);
        c += __popcll(__ballot(i < n && starts[min(i, n - 1)] <= at));
    }
    return c - 1;
}

constexpr int QUANT_PARTS = 2048;  // most workgroups of the quantizer kernels
// Totals of the quantizer's workgroups (sum g~, sum h~, sum |g~|), by a workgroup of 256 threads; every thread gets them.
__device__ __forceinline__ void sum_totals(const int64_t* __restrict__ part, int n_part, int64_t (&s)[3]) {
    __shared__ int64_t t[3][4];
    s[0] = s[1] = s[2] = 0;
    for (int i0 = 0; i0 < n_part; i0 += 4 * 256) {  // (four in flight)
        int64_t v[4][3];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            for (int k = 0; k < 3; ++k) v[u][k] = part[3 * min(i0 + 256 * u + (int)threadIdx.x, n_part - 1) + k];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            for (int k = 0; k < 3; ++k) s[k] += i0 + 256 * u + (int)threadIdx.x < n_part ? v[u][k] : 0;
    }
    for (int k = 0; k < 3; ++k) {
        for (int o = 32; o > 0; o >>= 1) s[k] += __shfl_xor(s[k], o);
        if ((threadIdx.x & 63) == 0) t[k][threadIdx.x >> 6] = s[k];
    }
    __syncthreads();
    for (int k = 0; k < 3; ++k) s[k] = t[k][0] + t[k][1] + t[k][2] + t[k][3];
}

constexpr int PART_GROUPS = 512;
// Passes over finished leaves gather and update 4 to 8 bytes per row, leaf by leaf, in places that lie about a cache line apart
// or further.  Their work is cut into parts of the row order (a leaf's list ascends), a multiple of 8 of them, and the
// workgroups of one part run side by side on one XCD: its L2 then serves all leaves' shares of a line after one fetch.
// A part is at most 2^17 rows up to 2^25 rows in all (then there are 256, of more rows each): 1 MB of (g, h) pairs, of which two to
// four parts in flight fit the 4 MB.
// Against 32 parts per leaf spread over all XCDs (and a separate copy of the row lists): 20 M rows in 511 leaves, refit and copy
// 430 -> 150 us, score update 635 -> 253 us (what is left is the rate of L2 requests, one per row and direction); 10.5 M
// rows in 255 leaves 179 -> 77 us; two leaves of 3 M rows 95 -> 11 us, which used to have 64 workgroups.
constexpr int REFIT_EXTRA = 256;  // most units of a part beyond one per leaf: large leaves are cut into several
inline int refit_parts(int64_t n_rows) {
    const int64_t p = 8 * ((n_rows + (1 << 20) - 1) >> 20);
    return p < 8 ? 8 : p > 256 ? 256 : (int)p;
}
inline int refit_extra(int64_t n_rows) {  // about 512 rows per unit where a leaf is large enough
    const int64_t x = n_rows / ((int64_t)refit_parts(n_rows) * 512);
    return x > REFIT_EXTRA ? REFIT_EXTRA : (int)x;
}
// Rows per thread of a segment of the batched partition (256 threads; the loads of a thread's rows are in flight
// together), and whether the left rows of PART_SUPER segments are summed up in one counter on the way.
//  - Up to 2^18 rows 2 rows per thread: segments of 2048 rows would leave most compute units without one (count + scatter
//    kernel per round on 10 k x 28 in ordered mode: 17.0 us with 8, 10.0 us with 2); above that 8, which spreads a
//    wavefront's fixed work per segment (1 M x 28: 10.8 us with 8, 14.6 us with 2).
//  - The counters save the scatter kernel a walk over all of a node's segments (2 KB per wavefront and million rows), but
//    their device-wide atomics lengthen the count kernel by about 2 us (1 M x 28: 7.9 us with, 6.1 us without).  Trees
//    with / without, matrix bound: 3.3 M x 28 907 / 887 us, 4 M 993 / 979 us, 4.7 M 1088 / 1079 us, 5.5 M 1198 / 1201 us, 6.2 M
//    1289 / 1302 us, 4 M x 100 1096 / 1077 us, 5.5 M x 100 1683 / 1687 us; not bound: 3.5 M x 60 1463 / 1482 us, 4.5 M x 60 1496 / 1519 us,
//    5.5 M x 20 1145 / 1154 us.  The lines lie where the two are level: between 4.7 and 5.5 M rows bound, below 3.5 M not bound.
inline int part_rows(int64_t n_rows) { return n_rows > ((int64_t)1 << 18) ? 8 : 2; }
inline bool part_supers(int64_t n_rows, bool bound) { return n_rows > ((int64_t)(bound ? 5 : 3) << 20); }
constexpr int PART_SUPER = 32;  // segments whose left rows are summed up in one counter
// Most nodes expanded in one round = most builds of a histogram launch (the leaf budget; the growth bookkeeping
// limits it to 658).  Kernels keep the first work item of every build / node in LDS and search there: a binary
// search through global memory costs a chain of dependent loads per work item.
constexpr int TABLE_MAX = 768;
// Largest leaf budget: 6 * 658 + 1 nodes may become known, and the growth bookkeeping (tree_plan_kernel) holds them in
// one workgroup's LDS, as 64 masks of 64 gain ranks and with 16-bit node ids.
constexpr int MAX_TREE_LEAVES = 658;

int set_error(qgbdt_ctx* ctx, int code, const char* fmt, ...);

#define QG_HIP(ctx, expr)                                                                      \
    do {                                                                                       \
        hipError_t e__ = (expr);                                                               \
        if (e__ != hipSuccess)                                                                 \
            return qgbdt::set_error(ctx, QGBDT_E_HIP, "%s failed: %s (%s:%d)", #expr,          \
                                    hipGetErrorString(e__), __FILE__, __LINE__);               \
    } while (0)

// launchers (each defined next to its kernels)
int launch_quantize(qgbdt_ctx* ctx, const float* g, const float* h, int64_t n, int bits_g, int bits_h,
                    uint64_t seed, uint32_t iteration, int rounding, int16_t* gh, float* delta_out,
                    int64_t* totals_out, float2* pairs_out);  // totals_out null: only the workgroups' totals (quantize_parts of them)
int quantize_parts(const float* g, const float* h, const int16_t* gh, int64_t n);
bool counting_build_ok(const qgbdt_ctx* ctx, const HistPlan& plan, const RowSource& rows);  // a launch of `plan` can count the round's rows itself
// Whether the histogram launches of a tree on row lists without gradient lists count the left rows (bound: there is a feature-major copy)
bool counts_rows(const qgbdt_ctx* ctx, const HistPlan& plan, const RowSource& rows, bool bound, int num_leaves);
// Segments that workgroup `block` of `grid` counts in a round of n_nodes nodes with first segments `starts` (n_segs in all):
// pairs of node and segment; returns their number, of which at most `room` are written
int64_t order_of_segments(const qgbdt_shape& s, bool bound, const int32_t* starts, int n_nodes, int n_segs, int block, int grid, int32_t* out, int64_t room);
HistPlan make_hist_plan(const qgbdt_shape& s, int bits_g, int bits_h, int acc_width, bool skew = false);
HistPlan make_hist_plan_for(const qgbdt_shape& s, int bits_g, int bits_h, int acc_width, int64_t rows, bool skew = false,
                            bool stream_ok = false);  // stream_ok: contiguous rows of a 16-byte aligned matrix
int64_t max_rows_for_width(int bits_g, int bits_h, int w);
int launch_begin_build(qgbdt_ctx* ctx, const HistPlan& plan, int64_t begin, int64_t count, int64_t* hist, int64_t n_words);
int launch_hist(qgbdt_ctx* ctx, const HistPlan& plan, const RowSource& rows, const IdxSet& idx, bool use_idx,
                bool flat_ok, const HistEntry* entries, const int32_t* table_counts, int64_t* hist_base,
                int64_t grid_items, const uint16_t* mfb = nullptr,
                int reduce_above = 0, const CountSource* count = nullptr);  // > 0: only builds of more row groups are added up by the reduce kernel
int launch_fill_zero(qgbdt_ctx* ctx, int64_t* p, int64_t n_words);
int launch_subtract(qgbdt_ctx* ctx, const int64_t* parent, const int64_t* child, int64_t* out, int64_t n);
// Best split of up to 2 * max_pairs histograms: candidates per (histogram, tile of features); `plan`: of the histogram launch
// whose slots the pairs refer to
int launch_scan_pairs(qgbdt_ctx* ctx, int64_t* hist_base, const ScanPair* pairs, const int32_t* n_items, int max_pairs,
                      const float* delta, int min_data, double min_sum_hess, FeatCand* cand, const uint16_t* mfb,
                      const HistPlan* plan, const RowMover* mover = nullptr);
int scan_candidates(const qgbdt_shape& s);  // candidates per scanned histogram
// candidates -> best splits, `stride` bytes apart from `out` on; step: growth state whose nodes' best splits are meant
int launch_reduce_items(qgbdt_ctx* ctx, const FeatCand* cand, const ScanPair* pairs, const int32_t* n_items, int max_items,
                        qgbdt_split* out, size_t stride, const StepState* step);
// stand-alone search in batches of `cap` histograms; scratch: pairs [(cap + 1) / 2], cand [cap][scan_candidates], n_items [1]
int run_find_best_splits(qgbdt_ctx* ctx, const int64_t* hist, int n_hists, const qgbdt_leafstat* stats,
                         const float* delta, int min_data, double min_sum_hess, qgbdt_split* out, int cap,
                         ScanPair* pairs, FeatCand* cand, int32_t* n_items);
int run_partition_rows(qgbdt_ctx* ctx, const uint8_t* bins, int32_t* row_idx, int64_t begin, int64_t count,
                       int feature, int bin, int64_t* n_left_out);
int launch_batch_partition_count(qgbdt_ctx* ctx, const RowSource& rows, const uint8_t* bins_t, bool ordered);
int launch_transpose_bins(qgbdt_ctx* ctx, const void* bins, void* out);
int launch_pad_bins(qgbdt_ctx* ctx, const void* bins, uint8_t* out, int pitch);
int launch_frequent_bins(qgbdt_ctx* ctx, const void* bins_t, uint16_t* mfb);
int launch_fix_frequent_bins(qgbdt_ctx* ctx, int64_t* hist, const int64_t* totals, const uint16_t* mfb);
int require_workspace(qgbdt_ctx* ctx);   // QGBDT_E_WORKSPACE unless a workspace block is set
int prepare_hist_kernels(qgbdt_ctx* ctx);  // once per context: dynamic-LDS limits of the kernels that exceed the default
int prepare_tree_kernels(qgbdt_ctx* ctx);
// !ordered: row ids and, with rows.gh_pos, packed gradients; `plan`: of the histogram launch that follows
int launch_batch_partition_scatter(qgbdt_ctx* ctx, const RowSource& rows, bool ordered, const HistPlan& plan);
int launch_refit(qgbdt_ctx* ctx, const float* g, const float* h, const int32_t* row_idx, const int64_t* leaf_begin,
                 const int64_t* leaf_count, int n_leaves, double* value_out);
// tree growth (leaves laid out; nothing happens while the tree is not finished): the row lists to the caller's, and the leaf values
int launch_gather_refit(qgbdt_ctx* ctx, const IdxSet& idx, uint32_t id_mask, int32_t* row_idx_out, const int32_t* n_leaves_dev, double* value_out);
int launch_logistic_gradients(qgbdt_ctx* ctx, const float* score, const float* label, int64_t n, float* g, float* h);
int launch_lambdarank_gradients(qgbdt_ctx* ctx, const float* score, const float* label, int64_t n, int group,
                                float* g, float* h);
// laid_out: by the tree that has just been grown (n_leaves: at most that many leaves)
int launch_update_scores(qgbdt_ctx* ctx, float* score, const int32_t* row_idx, const int64_t* leaf_begin,
                         const int64_t* leaf_count, const double* leaf_value, int n_leaves, bool laid_out, double lr);
int run_grow_tree(qgbdt_ctx* ctx, const uint8_t* bins, const float* g, const float* h,
                  const qgbdt_params* p, uint32_t iteration, const qgbdt_tree* out, int32_t* row_idx_out);

}  // namespace qgbdt
