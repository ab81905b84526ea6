// Device helpers of the split search shared by the stand-alone entry point and
// the tree-growing kernels.
#pragma once
#include "common.h"

namespace qgbdt {

// Two histograms to scan, in one record so that a workgroup of the split search needs a single load before it knows
// everything: `a` was built from rows (or is given), `b` is formed as parent - a first (or is given, or absent).  In tree
// growth they are the two children of a node; results are numbered 2 * pair + (0 or 1), `a` is number `a_item`.
struct ScanPair {
    int32_t slot_a, slot_b;  // histogram indices relative to the base pointer; slot_b < 0: no second histogram
    int32_t parent;          // >= 0: hist[slot_b] = hist[parent] - hist[slot_a] first
    int32_t a_item;
    int32_t item_start;      // first slot of a's row groups
    int32_t groups;          // > 0: a is the sum of that many slots, which the split search adds up; 0: it lies in hist[slot_a]
    int32_t merged;          // (groups > 0) hist[slot_a] holds what long row groups have merged already, to be added
    int32_t seg_start;       // (counting build) first segment of the parent's rows; n_rows of both totals is then the parent's
    qgbdt_leafstat stat[2];  // totals of a, b
};

__device__ __forceinline__ int64_t packed_g(int64_t w) { return w >> 32; }
__device__ __forceinline__ int64_t packed_h(int64_t w) { return w & 0xffffffffLL; }

// (G*dg)^2 / (2*H*dh), fp64, this operation order (Sec. 4.1 eq. (gain)); the
// translation unit is compiled without FMA contraction.
__device__ __forceinline__ double half_loss(int64_t G, int64_t H, double dg, double dh) {
    const double a = (double)G * dg;
    const double num = a * a;
    const double den = 2.0 * ((double)H * dh);
    return num / den;
}

// Left row count from the hessian share, rounded half up, exact integers.
__device__ __forceinline__ int64_t count_estimate(int64_t HL, int64_t Hs, int64_t n) {
    return (2 * HL * n + Hs) / (2 * Hs);
}

// Reduces the candidates of one leaf (F of them, one per tile of ascending features) to its best split: largest gain,
// ties to the lowest feature.  Called by all 64 lanes of one wavefront; lane 0
// writes the result.  estimate: with the left row count by the hessians; not in growth, which counts rows and whose
// pairs may hold the parent's number of rows (ScanPair::seg_start).
__device__ inline void reduce_features_wave(const FeatCand* cand, int F, const qgbdt_leafstat& st, qgbdt_split* out,
                                            int lane, bool estimate) {
    double bg = 0.0;
    int bf = -1;
    for (int f = lane; f < F; f += 64) {
        const FeatCand c = cand[f];
        if (c.bin >= 0 && (c.gain > bg)) { bg = c.gain; bf = f; }  // ascending f: strict > keeps the lowest
    }
    for (int o = 32; o > 0; o >>= 1) {
        const double og = __shfl_xor(bg, o);
        const int of = __shfl_xor(bf, o);
        if (of >= 0 && (bf < 0 || og > bg || (og == bg && of < bf))) { bg = og; bf = of; }
    }
    if (lane == 0) {
        qgbdt_split s;
        s.gain = 0.0; s.feature = -1; s.bin = -1;
        s.left_g = s.left_h = s.right_g = s.right_h = s.left_count = 0;
        if (bf >= 0) {
            const FeatCand c = cand[bf];
            s.gain = c.gain; s.feature = c.feature; s.bin = c.bin;
            s.left_g = packed_g(c.left); s.left_h = packed_h(c.left);
            s.right_g = st.sum_g - s.left_g; s.right_h = st.sum_h - s.left_h;
            if (estimate) s.left_count = count_estimate(s.left_h, st.sum_h, st.n_rows);
        }
        *out = s;
    }
}

// A histogram's totals, which the search has noted in its pair: both sides and which is which are read together.
struct ScanTotals {
    int64_t sum_g, sum_h;
};
__device__ __forceinline__ ScanTotals load_totals(const ScanPair* sp, int side) {
    const int a = sp->a_item;
    const int64_t g0 = sp->stat[0].sum_g, h0 = sp->stat[0].sum_h, g1 = sp->stat[1].sum_g, h1 = sp->stat[1].sum_h;
    return {a == side ? g0 : g1, a == side ? h0 : h1};
}

// The first four candidates of lane `sl` of a group of `sub` lanes (past the last one: that one again).
__device__ __forceinline__ void load_candidates(const FeatCand* cand, int F, int sl, int sub, FeatCand (&c)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) c[u] = cand[min(sl + u * sub, F - 1)];
}

// The same reduction by a group of `sub` consecutive lanes (a power of two, 64 at most; `sl` = lane inside
// the group), so that one wavefront serves 64 / sub leaves at a time.  c: the group's first candidates, loaded in advance.  The
// winner's candidate travels with the comparison: no load depends on another.  Every lane of the group returns the winner's gain and feature
// (feature < 0: no split).  (The count estimate is left out: growth counts rows, and a 64-bit division is a long chain.)
__device__ __forceinline__ void reduce_candidates(FeatCand (&c)[4], const FeatCand* cand, int F, const ScanTotals& st, qgbdt_split* out,
                                                  int sl, int sub, double& gain, int& feature) {
    double bg = 0.0;
    int bf = -1, bb = -1;  // (bf: the winner's feature)
    int64_t bl = 0;
    for (int f0 = sl;;) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {  // ascending features: strict > keeps the lowest
            const int f = f0 + u * sub;
            if (f < F && c[u].bin >= 0 && (c[u].gain > bg)) { bg = c[u].gain; bf = c[u].feature; bb = c[u].bin; bl = c[u].left; }
        }
        f0 += 4 * sub;
        if (f0 >= F) break;
        load_candidates(cand, F, f0, sub, c);
    }
    for (int o = sub >> 1; o > 0; o >>= 1) {
        const double og = __shfl_xor(bg, o);
        const int of = __shfl_xor(bf, o);
        const int ob = __shfl_xor(bb, o);
        const int64_t ol = __shfl_xor(bl, o);
        if (of >= 0 && (bf < 0 || og > bg || (og == bg && of < bf))) { bg = og; bf = of; bb = ob; bl = ol; }
    }
    if (sl == 0) {
        qgbdt_split s;
        s.gain = 0.0; s.feature = -1; s.bin = -1;
        s.left_g = s.left_h = s.right_g = s.right_h = s.left_count = 0;
        if (bf >= 0) {
            s.gain = bg; s.feature = bf; s.bin = bb;
            s.left_g = packed_g(bl); s.left_h = packed_h(bl);
            s.right_g = st.sum_g - s.left_g; s.right_h = st.sum_h - s.left_h;
        }
        *out = s;
    }
    gain = bg;  // (all lanes of the group hold the winner)
    feature = bf;
}

}  // namespace qgbdt
