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

// Part and unit of the calling wavefront (workgroups of four); false: none.  Consecutive workgroups go to the 8 XCDs in
// turn: the workgroups of a part are those of one XCD, and its parts follow each other.
__device__ __forceinline__ bool refit_unit_of(const int32_t* __restrict__ n_units, int blocks_per_part, int& part, int& u) {
    const int xcd = blockIdx.x & 7, s = blockIdx.x >> 3;
    part = s / blocks_per_part * 8 + xcd;
    u = __builtin_amdgcn_readfirstlane((s % blocks_per_part) * 4 + (int)(threadIdx.x >> 6));
    return u < *n_units;
}

}  // namespace qgbdt
