// Layout of finished leaves as units of equal work, for the kernels that pass over their rows.
#pragma once
#include "common.h"

namespace qgbdt {

struct LeafLayout {
    int64_t begin[MAX_TREE_LEAVES], count[MAX_TREE_LEAVES];
    int first[MAX_TREE_LEAVES + 1];  // first unit of a part
    int buf[MAX_TREE_LEAVES];
    int64_t wsum[16];
};

// Called by all 1024 threads of a workgroup with begin, count and buf of n (at most MAX_TREE_LEAVES) leaves in s, behind a barrier.
// A leaf gets one unit per part and, of `extra` further ones, its share by rows: at most n + extra in all.
__device__ __forceinline__ void layout_leaves(LeafLayout& s, int n, int max_leaves, int parts, int extra, RefitUnit* units,
                                              int2* leaves) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int64_t c = tid < n ? max(s.count[tid], (int64_t)0) : 0;
    const int64_t own = c;
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if (lane == 0) s.wsum[wave] = c;
    __syncthreads();
    int64_t total = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) total += s.wsum[k];
    const int mine = tid < n ? 1 + (total > 0 ? (int)(own * extra / total) : 0) : 0;
    int incl = mine;
    for (int o = 1; o < 64; o <<= 1) { const int u = __shfl_up(incl, o); if (lane >= o) incl += u; }
    __syncthreads();
    if (lane == 63) s.wsum[wave] = incl;
    __syncthreads();
    for (int k = 0; k < wave; ++k) incl += (int)s.wsum[k];
    if (tid < n) { s.first[tid] = incl - mine; leaves[tid] = make_int2(incl - mine, mine); }
    if (tid == n - 1) { s.first[n] = incl; leaves[max_leaves] = make_int2(incl, 0); }
    __syncthreads();
    for (int u = tid; u < s.first[n]; u += blockDim.x) {
        int lo = 0, hi = n - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s.first[mid] <= u) lo = mid; else hi = mid - 1;
        }
        RefitUnit r;
        r.begin = s.begin[lo]; r.count = max(s.count[lo], (int64_t)0); r.first = s.first[lo]; r.n = s.first[lo + 1] - s.first[lo];
        r.leaf = lo; r.buf = s.buf[lo];
        const int64_t pieces = (int64_t)parts * r.n;
        r.piece_rows = (r.count + pieces - 1) / pieces;
        units[u] = r;
    }
}

struct LeafList {
    const int64_t* begin;
    const int64_t* count;
    int n, extra;
};

// The layout for leaves that the caller lists, found by the wavefront that needs unit `u` of a part (false: none; uniform).  A
// launch of its own for the layout costs more than the search in every wavefront (the counts of the leaves, 64 at a time, twice):
// refit / score update of 10 k rows in 15 leaves 15.1 / 9.8 -> 11.6 / 7.4 us, of 3 M rows in 255 leaves 36.2 / 32.8 -> 33.3 / 29.2 us.
// A leaf's share of the further units goes by its count in blocks of 1024 rows, in 32 bits, which keeps the search short: the sum
// of 658 counts of at most 2^21 blocks fits, and three roundings to fp32 (2^-24 each) cannot carry a share that is taken 2^-20
// smaller above the exact one, so there are n + extra units at most.
__device__ __forceinline__ bool find_unit(const LeafList& list, int parts, int u, RefitUnit& r) {
    const int n = list.n, lane = threadIdx.x & 63;
    auto blocks = [](int64_t count) { return (int)min(max(count, (int64_t)0) >> 10, (int64_t)1 << 21); };
    int total = 0;
    for (int t = lane; t < n; t += 64) total += blocks(list.count[t]);
    total = wave_sum(total);
    const float share = total > 0 ? (float)list.extra * (1.0f - 0x1p-20f) / (float)total : 0.0f;
    int base = 0;
    for (int t0 = 0; t0 < n; t0 += 64) {
        const int t = t0 + lane, at = min(t, n - 1);
        const int64_t begin = list.begin[at], count = max(list.count[at], (int64_t)0);
        const int mine = t < n ? 1 + (int)((float)blocks(count) * share) : 0;
        const int incl = base + wave_prefix(mine);
        const unsigned long long found = __ballot(incl > u);
        if (found) {
            const int src = __ffsll((long long)found) - 1;
            r.leaf = t0 + src; r.buf = 0;
            r.n = __builtin_amdgcn_readlane(mine, src);
            r.first = __builtin_amdgcn_readlane(incl, src) - r.n;
            r.begin = readlane64(begin, src);
            r.count = readlane64(count, src);
            const int pieces = parts * r.n;  // (a quotient below 2^48 that is no integer is rounded to none in fp64)
            r.piece_rows = (int64_t)((double)(r.count + pieces - 1) / (double)pieces);
            return true;
        }
        base = __builtin_amdgcn_readlane(incl, 63);
    }
    return false;
}

// Part and unit of the calling wavefront (workgroups of four).  Consecutive workgroups go to the 8 XCDs in
// turn: the workgroups of a part are those of one XCD, and its parts follow each other.
__device__ __forceinline__ void refit_unit_of(int blocks_per_part, int& part, int& u) {
    const int xcd = blockIdx.x & 7, s = blockIdx.x >> 3;
    part = s / blocks_per_part * 8 + xcd;
    u = __builtin_amdgcn_readfirstlane((s % blocks_per_part) * 4 + (int)(threadIdx.x >> 6));
}

}  // namespace qgbdt
