// Sibling subtraction and best-split search over integer histograms (threshold
// enumeration of Sec. 3 with the quantized gain of Sec. 4.1 eq. (gain)).
// Integer prefix sums over the packed words, fp64 gain; compiled with FMA
// contraction off so that the gain is evaluated operation by operation.
#include <algorithm>
#include <type_traits>

#include "partition_device.h"

namespace qgbdt {

__global__ void subtract_kernel(const int64_t* __restrict__ parent, const int64_t* __restrict__ child,
                                int64_t* out, int64_t n) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    // a bin's child sums never exceed its parent's, so the packed words subtract field by field
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) out[i] = parent[i] - child[i];
}

int launch_subtract(qgbdt_ctx* ctx, const int64_t* parent, const int64_t* child, int64_t* out, int64_t n) {
    int blocks = (int)((n + 255) / 256);
    if (blocks > 1024) blocks = 1024;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(subtract_kernel, dim3(blocks), dim3(256), 0, ctx->stream, parent, child, out, n);
    QG_HIP(ctx, hipGetLastError());
    return QGBDT_OK;
}

__global__ void scan_pairs_from_stats_kernel(const qgbdt_leafstat* stats, int n, ScanPair* pairs, int32_t* n_items) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (2 * t < n) {
        ScanPair sp;
        sp.slot_a = 2 * t; sp.slot_b = 2 * t + 1 < n ? 2 * t + 1 : -1; sp.parent = -1; sp.a_item = 0;
        sp.item_start = 0; sp.groups = 0; sp.merged = 0; sp.seg_start = 0;
        sp.stat[0] = stats[2 * t]; sp.stat[1] = stats[min(2 * t + 1, n - 1)];
        pairs[t] = sp;
    }
    if (t == 0) *n_items = n;
}

// Largest unsigned value of the lanes with DPP moves (no LDS traffic); uniform.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#define QG_DPP(ctrl, rmask) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rmask, 0xf, false))
    QG_DPP(0x111, 0xf); QG_DPP(0x112, 0xf); QG_DPP(0x114, 0xf); QG_DPP(0x118, 0xf);  // row_shr: lane 15 of a row has its maximum
    QG_DPP(0x142, 0xa); QG_DPP(0x143, 0xc);                                          // row_bcast:15, row_bcast:31
#undef QG_DPP
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Where the row groups of a launch have left their local bins.
struct SlotSource {
    const unsigned char* partials;
    int32_t elementwise;  // slots of the element-wise kernel: the pitch is the tile's own width
    int32_t acc_width, hshift, ft, ftp, n_tiles, slot_bytes, pad16;
};

// Sum over a build's slots of the words of feature f and bins b .. b + KB - 1, as packed 32|32 words.
template <int W, int KB>
__device__ __forceinline__ void sum_slots(const SlotSource& s, int item_start, int groups, int b, int nb, int f, int F, int64_t (&out)[KB]) {
    using word = typename std::conditional<W == 16, uint32_t, int64_t>::type;
    const int tile = f / s.ft, fl = f - tile * s.ft;
    const int pitch = s.elementwise ? min(s.ft, F - tile * s.ft) : s.ftp;
    const int col = fl + (s.pad16 ? 4 * (fl >> 4) : 0);
    const size_t stride = (size_t)s.n_tiles * (size_t)s.slot_bytes;
    const unsigned char* p = s.partials + ((size_t)item_start * s.n_tiles + tile) * (size_t)s.slot_bytes;
    uint32_t off[KB];  // of the bins (past the last one: the last one again, not used)
#pragma unroll
    for (int k = 0; k < KB; ++k) off[k] = (uint32_t)(min(b + k, nb - 1) * pitch + col) * (uint32_t)sizeof(word);
    const uint32_t mask = (1u << s.hshift) - 1u;
    int32_t g[KB] = {};
    uint32_t h[KB] = {};
    int64_t w64[KB] = {};
    constexpr int U = (W == 16 ? 32 : 16) / KB < 8 ? (W == 16 ? 32 : 16) / KB : 8;  // slots whose loads are in flight together
    for (int i = 0; i < groups; i += U) {
        word x[U][KB];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned char* q = p + (size_t)min(i + u, groups - 1) * stride;
#pragma unroll
            for (int k = 0; k < KB; ++k) x[u][k] = *reinterpret_cast<const word*>(q + off[k]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < KB; ++k) {
                const word v = i + u < groups ? x[u][k] : (word)0;
                if (W == 16) { g[k] += (int32_t)(uint32_t)v >> s.hshift; h[k] += (uint32_t)v & mask; }
                else w64[k] += (int64_t)v;
            }
    }
#pragma unroll
    for (int k = 0; k < KB; ++k) out[k] = W == 16 ? (int64_t)g[k] * 4294967296LL + (int64_t)h[k] : w64[k];
}

// The winner of a set of candidates, one per lane: largest gain (> 0), ties to the lowest `code` (feature, then bin).  The
// lane's index is returned (uniform), -1 if no lane has a gain.
// (Gains are not negative, so their bits order like unsigned integers: upper halves first, then lower ones.)
__device__ __forceinline__ int wave_argmax(double gain, uint32_t code) {
    const uint64_t bits = (uint64_t)__double_as_longlong(gain);
    const uint32_t hi = (uint32_t)(bits >> 32), lo = (uint32_t)bits;
    const uint32_t mh = wave_max_u32(hi);
    unsigned long long m = __ballot(hi == mh);
    if (m & (m - 1ull)) {
        const uint32_t ml = wave_max_u32(hi == mh ? lo : 0u);
        m = __ballot(hi == mh && lo == ml);
        if (mh == 0u && ml == 0u) return -1;
    }
    int win = __ffsll((long long)m) - 1;
    uint32_t low = (uint32_t)__builtin_amdgcn_readlane((int)code, win);
    for (m &= m - 1ull; m; m &= m - 1ull) {  // (equal gains are rare)
        const int l = __ffsll((long long)m) - 1;
        const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)code, l);
        if (c < low) { low = c; win = l; }
    }
    return win;
}

// Matrices whose tiles are spread over all XCDs when there are few pairs, instead of a whole pair on one: those of which a single
// pair has more wavefronts than the 32 compute units of an XCD run at full speed side by side.  From 32 pairs on the XCDs'
// shares differ by a quarter at most.  Calls of the stand-alone search with whole pairs / spread: one histogram of 2000 features,
// 255 bins 51.9 / 17.8 us, 17 of them 98 / 65 us, two of 900 features, 300 bins 47.7 / 16.0 us, 18 of 2000 features, 63 bins
// 24.6 / 20.7 us; trees of 40 k x 2000, 255 bins 1057 / 854 us, of 400 k x 2000, 63 bins 1225 / 1195 us.  Below the line a launch
// of a tree would lose 0.3 to 0.6 us to the second order of the work and gain nothing (464 k x 90, 2 M x 40 of 600 bins).
__host__ __device__ __forceinline__ bool scan_spread(int n_tiles, int waves_per_tile) {
    return (int64_t)n_tiles * waves_per_tile > 256;
}
constexpr int SPREAD_PAIRS = 32;

// Best split per tile of T features, for two histograms at a time, in tree growth the two children of a node.  The child
// that was built from rows comes from its row groups' slots (or, when a reduce kernel has summed
// them up, from the pool), its sibling is parent - child; both are written to the pool on the way.  A thread owns one feature
// and KB consecutive bins of both histograms, a wavefront T features x 64 / T such segments: integer prefix sums (the
// fields cannot overflow: every prefix is bounded by the leaf's totals) over the thread's bins, over the wavefront's segments and,
// through LDS, over the wavefronts; then the fp64 gain of every threshold and the arg-max over the workgroup.
// Bound by the instructions of a threshold (about 130, most of them two IEEE fp64 divisions) for wide matrices, by the
// chain of latencies for narrow ones: one record per pair, the sums of slots and the parent's words loaded together, and
// no branches between the thresholds, so that their dependent operations interleave.
// Measured per launch with the reduce kernel's launch in front of it, against one workgroup per feature (or per 16 features and
// 1024 threads) and histogram behind a full reduction: 1 M x 28, 255 bins 15.0 -> 12.6 us; 464 k x 90 28.1 -> 18.8 us;
// 2 M x 40, 600 bins 38.1 -> 23.8 us; 400 k x 2000, 63 bins (and one launch less) 46.7 -> 28.6 us; 20 M x 200 34.1 -> 25.4 us.
template <int T, int NB64, int KB, bool SPREAD, int R>  // features per workgroup; bins, in units of 64; bins per thread; scan_spread; R > 0: moves rows too
__global__ __launch_bounds__(64 * T * NB64 / KB) void scan_pair_kernel(int64_t* hist_base, const ScanPair* __restrict__ pairs,
                                                                  const int32_t* __restrict__ n_items_ptr, int max_pairs, SlotSource slots,
                                                                  int F, int nb, const float* __restrict__ delta, int min_data,
                                                                  double min_sum_hess, FeatCand* __restrict__ cand_base,
                                                                  const uint16_t* __restrict__ mfb, typename std::conditional<(R > 0), RowMover, int>::type mover) {
    int n_blocks = (int)gridDim.x;
    if constexpr (R > 0) {
        n_blocks = mover.scan_blocks;
        if ((int)blockIdx.x >= n_blocks) { move_rows<R>(mover, (int)blockIdx.x - n_blocks, (int)gridDim.x - n_blocks); return; }
    }
    constexpr int NW = T * NB64 / KB;  // wavefronts
    const int n_items = *n_items_ptr;
    const double dg = (double)delta[0], dh = (double)delta[1];
    const int n_ft = (F + T - 1) / T, n_pairs = (n_items + 1) / 2;
    // Consecutive workgroups go round-robin to the XCDs: the tiles of a pair, which share cache lines, stay on one.  Few pairs of
    // a wide matrix are spread: every XCD takes an eighth of the tiles of all pairs, consecutive ones.
    const int xcd = blockIdx.x & 7, sid = blockIdx.x >> 3;
    const bool spread = SPREAD && n_pairs < SPREAD_PAIRS;
    const int n_work = spread ? n_pairs * n_ft : 0, share = (n_work + 7) >> 3;
    const int64_t W = (int64_t)F * nb;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int fl = threadIdx.x % T, b0 = (int)threadIdx.x / T * KB;
    __shared__ int64_t s_sum[2][NW][T];   // a wavefront's bins of a feature
    __shared__ FeatCand s_cand[2][NW];
    const int t0 = (sid / n_ft) * 8 + xcd;
    int tile = sid % n_ft, w = sid;
    ScanPair sp = pairs[min(t0, max_pairs - 1)];  // (in flight together with the number of items)
    for (int t = t0;; t += n_blocks / (8 * n_ft) * 8) {
        if (spread) {
            const int i = xcd * share + w;
            if (w >= share || i >= n_work) break;
            t = i / n_ft; tile = i - t * n_ft;
            w += n_blocks >> 3;
            sp = pairs[t];
        } else {
            if (t >= n_pairs) break;
            if (t != t0) sp = pairs[t];
        }
        const int f = tile * T + fl;
        const bool has_b = sp.slot_b >= 0;
        if constexpr (R > 0) {  // the children's rows: left ones by segment
            const int count = (int)sp.stat[0].n_rows, n_seg = (count + 256 * R - 1) / (256 * R);
            const int32_t* c = mover.seg_counts + sp.seg_start;
            int nl = 0;
            for (int k = 0; k < n_seg; k += 4 * 64) {
                int x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = c[min(k + 64 * u + lane, n_seg - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) nl += k + 64 * u + lane < n_seg ? x[u] : 0;
            }
            nl = wave_sum(nl);
            sp.stat[0].n_rows = sp.a_item ? count - nl : nl;  // (the built child comes first)
            sp.stat[1].n_rows = sp.a_item ? nl : count - nl;
        }
        const int64_t at = (int64_t)b0 * F + f;  // histograms are [bin][feature]
        int64_t v[2][KB] = {};                    // words, then inclusive prefix sums
        if (f < F && b0 < nb) {
            int64_t* const pa = hist_base + (int64_t)sp.slot_a * W + at;
            if (has_b) {
                const int64_t* p = hist_base + (int64_t)(sp.parent >= 0 ? sp.parent : sp.slot_b) * W + at;
#pragma unroll
                for (int k = 0; k < KB; ++k) if (b0 + k < nb) v[1][k] = p[(int64_t)k * F];
            }
            if (sp.groups > 0) {
                if (slots.acc_width == 16) sum_slots<16, KB>(slots, sp.item_start, sp.groups, b0, nb, f, F, v[0]);
                else sum_slots<32, KB>(slots, sp.item_start, sp.groups, b0, nb, f, F, v[0]);
            }
#pragma unroll
            for (int k = 0; k < KB; ++k) {
                if (b0 + k >= nb) v[0][k] = 0;
                else if (sp.groups == 0 || sp.merged) v[0][k] += pa[(int64_t)k * F];
            }
            if (sp.groups > 0) {
#pragma unroll
                for (int k = 0; k < KB; ++k) if (b0 + k < nb) pa[(int64_t)k * F] = v[0][k];
            }
            if (sp.parent >= 0) {
                int64_t* const pb = hist_base + (int64_t)sp.slot_b * W + at;
#pragma unroll
                for (int k = 0; k < KB; ++k) if (b0 + k < nb) { v[1][k] -= v[0][k]; pb[(int64_t)k * F] = v[1][k]; }
            }
        }
        int64_t before[2];  // the feature's bins in front of this thread's
#pragma unroll
        for (int side = 0; side < 2; ++side) {
#pragma unroll
            for (int k = 1; k < KB; ++k) v[side][k] += v[side][k - 1];
            int64_t incl = v[side][KB - 1];
#pragma unroll
            for (int o = T; o < 64; o <<= 1) {
                const int64_t u = __shfl_up(incl, o);
                if (lane >= o) incl += u;
            }
            before[side] = incl - v[side][KB - 1];
            if (lane >= 64 - T) s_sum[side][wave][fl] = incl;
        }
        __syncthreads();
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const int64_t Gs = sp.stat[side].sum_g, Hs = sp.stat[side].sum_h, n = sp.stat[side].n_rows;
            int64_t off = before[side], missing = 0;
            int mb = 0xffff;
#pragma unroll
            for (int w = 0; w < NW - 1; ++w) off += w < wave ? s_sum[side][w][fl] : 0;
            if (mfb != nullptr && f < F) {
                // The histogram kernels may have left out the feature's most frequent bin: the entry is then 0 and
                // what is missing from the feature's sum over all bins -- the leaf's totals are known -- belongs to
                // that bin.  (Nothing is missing when the bin was accumulated.)
                mb = mfb[f];
                if (mb != 0xffff) {
                    missing = Gs * 4294967296LL + Hs;
#pragma unroll
                    for (int w = 0; w < NW; ++w) missing -= s_sum[side][w][fl];
                }
            }
            // count_estimate(HL, Hs, n) = floor((2 HL n + Hs) / (2 Hs)) >= min_data, and <= n - min_data, without
            // the division (2 HL n < 2^64: the fields and row counts have 32 and 31 bits)
            const uint64_t n2 = 2ull * (uint64_t)n, uH = (uint64_t)Hs;
            const uint64_t lo_lim = min_data > 0 ? (2ull * (uint64_t)min_data - 1ull) * uH : 0ull;
            const uint64_t hi_lim = min_data <= 0 ? ~0ull : (n + 1 > (int64_t)min_data) ? (2ull * (uint64_t)(n - min_data + 1) - 1ull) * uH : 0ull;
            const double parent = half_loss(Gs, Hs, dg, dh);
            double gain = 0.0;
            int bin = 0;
            int64_t left = 0;
#pragma unroll
            for (int k = 0; k < KB; ++k) {  // ascending bins: strict > keeps the lowest
                int64_t pre = v[side][k] + off;
                if (mfb != nullptr && b0 + k >= mb) pre += missing;
                const int32_t GL = (int32_t)(pre >> 32);
                const uint32_t HL = (uint32_t)pre;
                const int64_t GR = Gs - GL, HR = Hs - (int64_t)HL;
                const uint64_t x = (uint64_t)HL * n2;
                const double hl = (double)HL * dh, hr = (double)HR * dh;
                const double al = (double)GL * dg, ar = (double)GR * dg;
                const double gn = (al * al) / (2.0 * hl) + (ar * ar) / (2.0 * hr) - parent;
                const bool ok = (f < F) & (b0 + k + 1 < nb) & (HL > 0u) & (HR > 0) & (x >= lo_lim) & (x < hi_lim) &
                                !(hl < min_sum_hess) & !(hr < min_sum_hess) & (gn > gain);
                gain = ok ? gn : gain; bin = ok ? b0 + k : bin; left = ok ? pre : left;
            }
            const int win = wave_argmax(gain, ((uint32_t)fl << 16) | (uint32_t)bin);
            if (lane == (win < 0 ? 0 : win)) {
                FeatCand fc;
                fc.gain = win < 0 ? 0.0 : gain; fc.left = left; fc.bin = win < 0 ? -1 : bin; fc.feature = f;
                s_cand[side][wave] = fc;
            }
        }
        __syncthreads();
        if (wave < 2 && NW > 1 ? true : wave == 0) {  // the tile's best: one wavefront per histogram (both by the only one)
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                if (NW > 1 && side != wave) continue;
                const FeatCand fc = s_cand[side][min(lane, NW - 1)];
                const int win = wave_argmax(lane < NW && fc.bin >= 0 ? fc.gain : 0.0, ((uint32_t)(fc.feature - tile * T) << 16) | (uint32_t)fc.bin);
                const int item = 2 * t + (side ^ sp.a_item);
                if (lane == (win < 0 ? 0 : win) && (side == 0 || has_b)) cand_base[(int64_t)item * n_ft + tile] = fc;
            }
        }
        __syncthreads();  // (s_sum and s_cand are reused)
    }
}

// Candidates (n_cand per histogram, one per tile of ascending features) -> best split of every scanned histogram, one
// wavefront per histogram.
__global__ __launch_bounds__(256) void reduce_items_kernel(const FeatCand* __restrict__ cand_base,
                                                           const ScanPair* __restrict__ pairs,
                                                           const int32_t* __restrict__ n_items_ptr, int n_cand,
                                                           unsigned char* out, int64_t stride, const StepState* step) {
    const int n_items = *n_items_ptr;
    const int first = step ? step->n_nodes - n_items : 0;  // tree growth: the histograms are those of the newest nodes
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int item = blockIdx.x * 4 + wave; item < n_items; item += gridDim.x * 4) {
        const ScanPair* sp = &pairs[item >> 1];
        reduce_features_wave(cand_base + (int64_t)item * n_cand, n_cand, sp->stat[sp->a_item == (item & 1) ? 0 : 1],
                             reinterpret_cast<qgbdt_split*>(out + (int64_t)(first + item) * stride), lane, step == nullptr);
    }
}

int launch_reduce_items(qgbdt_ctx* ctx, const FeatCand* cand, const ScanPair* pairs, const int32_t* n_items, int max_items,
                        qgbdt_split* out, size_t stride, const StepState* step) {
    int gr = (max_items + 3) / 4;
    if (gr > 256) gr = 256;
    hipLaunchKernelGGL(reduce_items_kernel, dim3(gr), dim3(256), 0, ctx->stream, cand, pairs, n_items,
                       scan_candidates(ctx->shape), reinterpret_cast<unsigned char*>(out), (int64_t)stride, step);
    QG_HIP(ctx, hipGetLastError());
    return QGBDT_OK;
}

// Features per tile of the split search: 16 (whole cache lines of the [bin][feature] histograms) for very wide matrices of
// up to 256 bins, four or two for the others, whose few histograms of a round would leave compute units idle otherwise
// (trees with tiles of 16 / of 4: 464 k x 90 775 / 745 us, 200 k x 136 968 / 897 us, 20 M x 200 14.9 / 14.7 ms).
static int scan_tile_features(const qgbdt_shape& s) { return s.n_bins > 256 ? 2 : s.n_features >= 256 ? 16 : 4; }
int scan_candidates(const qgbdt_shape& s) {
    const int T = scan_tile_features(s);
    return (s.n_features + T - 1) / T;
}

int launch_scan_pairs(qgbdt_ctx* ctx, int64_t* hist_base, const ScanPair* pairs, const int32_t* n_items, int max_pairs,
                      const float* delta, int min_data, double min_sum_hess, FeatCand* cand, const uint16_t* mfb,
                      const HistPlan* plan, const RowMover* mover) {
    const int F = ctx->shape.n_features, nb = ctx->shape.n_bins;
    const int n_ft = scan_candidates(ctx->shape);
    SlotSource src{};
    if (plan) {
        src.partials = static_cast<const unsigned char*>(ctx->hist_partials);
        src.acc_width = plan->two_level ? 32 : plan->acc_width; src.hshift = plan->hshift; src.ft = plan->ft; src.ftp = plan->ftp;
        src.n_tiles = plan->n_tiles; src.slot_bytes = plan->slot_bytes; src.pad16 = plan->pad16;
        src.elementwise = plan->bytewise;
    }
    // one workgroup per (tile, pair) up to about 4096 of them, pairs in multiples of 8 (one per XCD)
    int64_t lanes = max_pairs, most = 4096 / n_ft;
    if (most < 8) most = 8;
    if (lanes > most) lanes = most;
    lanes = (lanes + 7) / 8 * 8;
    // (where every number of pairs up to max_pairs is spread, no more than there are tiles)
#define QG_SCAN_R(T_, N_, K_, S_, R_, M_, X_)                                                                           \
    hipLaunchKernelGGL((scan_pair_kernel<T_, N_, K_, S_, R_>), dim3((unsigned)((lanes * n_ft + 7) / 8 * 8 + (X_))),     \
                       dim3(64 * T_ * N_ / K_), 0, ctx->stream, hist_base, pairs, n_items, max_pairs, src, F, nb,       \
                       delta, min_data, min_sum_hess, cand, mfb, M_)
#define QG_SCAN_S(T_, N_, K_, S_)                                                                                       \
    do {                                                                                                                \
        if (!mover) { QG_SCAN_R(T_, N_, K_, S_, 0, 0, 0); break; }                                                      \
        RowMover mv = *mover;                                                                                           \
        mv.scan_blocks = (int)((lanes * n_ft + 7) / 8 * 8);                                                             \
        const int movers = (int)std::min<int64_t>(2048, ((int64_t)ctx->max_seg * 4 + T_ * N_ / K_ - 1) / (T_ * N_ / K_)) + 1; \
        if (ctx->seg_rows == 256 * 8) QG_SCAN_R(T_, N_, K_, S_, 8, mv, movers);                                         \
        else QG_SCAN_R(T_, N_, K_, S_, 2, mv, movers);                                                                  \
    } while (0)
#define QG_SCAN(T_, N_, K_)                                                                                             \
    do {                                                                                                                \
        if (scan_spread(n_ft, T_ * N_ / K_)) {                                                                          \
            if (max_pairs < SPREAD_PAIRS && max_pairs < lanes) lanes = max_pairs;                                       \
            QG_SCAN_S(T_, N_, K_, true);                                                                                \
        } else QG_SCAN_S(T_, N_, K_, false);                                                                            \
    } while (0)
    // (bins per thread: few for narrow matrices, whose workgroups do not fill the chip; 1 M x 28 10.0 us per launch with four,
    // 9.7 us with two)
    if (nb > 512) QG_SCAN(2, 16, 4);
    else if (nb > 256) QG_SCAN(2, 8, 2);
    else if (scan_tile_features(ctx->shape) == 16) {
        if (nb <= 64) QG_SCAN(16, 1, 4);
        else if (nb <= 128) QG_SCAN(16, 2, 4);
        else QG_SCAN(16, 4, 4);
    } else if (nb <= 64) QG_SCAN(4, 1, 1);
    else if (nb <= 128) QG_SCAN(4, 2, 1);
    else if (F >= 64) QG_SCAN(4, 4, 4); else QG_SCAN(4, 4, 2);
#undef QG_SCAN
#undef QG_SCAN_S
#undef QG_SCAN_R
    QG_HIP(ctx, hipGetLastError());
    return QGBDT_OK;
}

// Stand-alone search over n_hists contiguous histograms, in batches of the tables it is given.
int run_find_best_splits(qgbdt_ctx* ctx, const int64_t* hist, int n_hists, const qgbdt_leafstat* stats,
                         const float* delta, int min_data, double min_sum_hess, qgbdt_split* out, int cap,
                         ScanPair* pairs, FeatCand* cand, int32_t* n_items) {
    const int64_t W = (int64_t)ctx->shape.n_features * ctx->shape.n_bins;
    for (int h0 = 0; h0 < n_hists; h0 += cap) {
        const int n = (n_hists - h0 < cap) ? (n_hists - h0) : cap, np = (n + 1) / 2;
        hipLaunchKernelGGL(scan_pairs_from_stats_kernel, dim3((np + 63) / 64), dim3(64), 0, ctx->stream, stats + h0, n, pairs, n_items);
        int rc = launch_scan_pairs(ctx, const_cast<int64_t*>(hist) + h0 * W, pairs, n_items, np, delta, min_data, min_sum_hess,
                                   cand, nullptr, nullptr);
        if (rc != QGBDT_OK) return rc;
        rc = launch_reduce_items(ctx, cand, pairs, n_items, n, out + h0, sizeof(qgbdt_split), nullptr);
        if (rc != QGBDT_OK) return rc;
    }
    return QGBDT_OK;
}

}  // namespace qgbdt
