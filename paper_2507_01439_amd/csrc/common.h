// Internal declarations shared by the HIP sources of libturboreg (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/turboreg.h"

namespace tr {

constexpr int kSc2Tile = 256;     // SC2 work-list tile edge (four 128 x 128 output tiles); npad is a multiple
constexpr int kHistGroups = 8;    // SC2 tiles add their weight histograms into this many copies per pair
constexpr int kCompatTile = 128;  // tile edge of the compatibility list
constexpr int kCompatMinRows = 8; // fewest rows of a tile one work item takes (Work::compat_rows)
constexpr int kRowsPerItem = 4;   // rows per work item of the pivot scans (one per wave)
constexpr int kPrepRows = 256;    // rows per work item of the prep / feature kernels
constexpr int kScoreHyp = 64;     // hypotheses per scoring work item (four per thread)
constexpr int kScorePts = 256;    // points per scoring work item (staged in LDS)
// Counters that many workgroups update with device-scope atomics are spread out: same-address
// device atomics are served one after another, so one shared counter serialises the stage.
constexpr int kCollectRegions = 8; // pivot collection: one pool region and counter per XCD
constexpr int kHypGroup = 32;     // clique-search items per first-level ticket
constexpr int kTickLine = 32;     // int32 per counter: one counter per 128-byte line
constexpr int kTickHyp0 = kCollectRegions;      // first clique-search group ticket
constexpr int kFusedPool = 512;   // learned pools up to this size are reordered inside the hypothesis kernel

// Work-list stages whose per-pair item counts depend on N_b; each has a
// prefix array of B+1 entries in Work::pre, over the pairs in cost order.
enum Stage { kPrep = 0, kCompat, kSc2, kSp, kCollect, kRowBlk, kScore, kNumPrefix };
// Rows of Work::pre after the stage prefixes: the cost order (slot -> pair), its inverse.
constexpr int kOrderRow = kNumPrefix, kSlotRow = kNumPrefix + 1, kPreRows = kNumPrefix + 2;

struct PairDesc {
    int32_t n;        // matches in this pair (0 when the pair is invalid)
    int32_t npad;     // n rounded up to kSc2Tile
    int32_t pt_off;   // first match of this pair in src/dst
    int32_t kpiv;     // pivots to select: min(k1 or pool, n(n-1)/2)
    int64_t c_off;    // entry offset of this pair in the C arena (npad x npad bits: c_off / 8 bytes)
    int64_t g_off;    // element offset of this pair's G in the G arena (npad x npad uint16)
};

// Per-pair scalars written by the kernels.
struct PairState {
    int32_t status;     // tr_status
    int32_t nonfinite;  // 1 if any coordinate is NaN/Inf (summed from the compatibility tiles)
    int32_t n_boundary;
    int32_t n_edges;
    int32_t alpha;      // weight of the last pivot (the K-th largest, Eq. 4)
    int32_t c_gt;       // edges heavier than alpha (all selected)
    int32_t m_eq;       // edges of weight alpha to take, in lexicographic order
    int32_t fallback;   // learned scores were not finite
    int32_t fast;       // every pair of weight >= alpha fits the pivot pool: collected unordered, then sorted
    int32_t ncand;      // keys the sort ranks (fast: c_gt + all ties; else K)
    int32_t done;       // ticket groups of the clique-search stage that have finished this pair
};

struct Plan {
    int32_t B;
    int32_t total[kNumPrefix];
    int32_t sp_tile;        // tile edge of the SC2 bit-count kernel, 0: every tile takes the product
    int32_t compat_rows;    // rows of a compatibility tile per work item: 8, 16, 32 or 128
    int32_t sc2_split[9];   // SC2 items [sc2_split[x], sc2_split[x+1]) go to XCD x: equal modelled cost
};

// Device views passed to every kernel.
struct Work {
    const float *src, *dst;
    const PairDesc *pairs;
    PairState *state;
    const Plan *plan;
    const int32_t *pre;       // kPreRows x (max_batch + 1): per stage, the first item of the pair in
                              // each slot of the cost order (largest pairs first); then the order
                              // (slot -> pair) and its inverse (pair -> slot)
    int32_t pre_stride;       // max_batch + 1
    int32_t n1;               // N of a single-pair call (its plan is computed in registers), 0 for a batch
    int32_t max_n;            // per-pair row stride of the per-row arenas
    int32_t k1, k2, pool;     // pool = plain pivots selected (k1, or pool_factor*k1 in learned mode)
    int32_t H;                // k1 * k2 hypotheses per pair
    int32_t graph;
    int32_t sc2_super;        // SC2 tile walk: super-tile side in output tiles (launch configuration)
    int32_t sp_tile;          // the same for a single-pair call (sc2_sparse_edge)
    int32_t sp_cap;           // it takes tiles of at most so many edges per 256 x 256 entries (launch configuration)
    int32_t *sp_list;         // the tiles it left to the dense kernel: their number, its next tile, its list
                              // items; null where it is not launched
    float tau, theta;
    uint8_t *C;               // C arena, one bit per entry: per pair npad x npad bits in blocks of 128 columns,
                              // [column / 128][row][16 bytes] (bit c % 8 of byte (c % 128) / 8); offset c_off / 8
    uint16_t *G;              // G arena
    int32_t *ghist;           // max_batch x kHistGroups x hist_stride weight histograms (filled by the SC2 epilogue)
    int32_t hist_stride;      // max_n rounded up to 8 (16-byte aligned copies)
    uint16_t *segmax;         // per pair npad x npad / 64 from g_off / 64: the maximum of G over the pairs i < j of row
                              // i in each 64-column segment (order: part_at; written by the SC2 kernels)
    int32_t compat_rows;      // the same for a single-pair call (compat_item_rows)
    uint32_t *cnt_part;       // per compatibility work item: edges (15 bits), boundary pairs << 15, non-finite
                              // input << 30
    int32_t *rowcnt;          // max_batch x max_n: pairs of weight alpha per row (ordered path)
    uint64_t *rowseg;         // max_batch x max_n: bit s set if the row's s-th 512-column segment (counted
                              // from its first column j > i) holds a pair of weight alpha (ordered path)
    int32_t *blkcnt;          // max_batch x nblk: pairs of weight alpha per block of kRowsPerItem rows
    int32_t nblk_stride;      // blocks of kRowsPerItem rows per pair (for max_n)
    uint64_t *cand;           // max_batch x kCollectRegions x pool_cap selection candidates (sort keys); the
                              // ordered path writes region 0 only
    int32_t *tick;            // max_batch x tick_stride counters, kTickLine apart: kCollectRegions collection
                              // counters, then one ticket per group of kHypGroup clique-search items
    int32_t tick_stride;
    uint64_t *hyp_rec;        // max_batch x rec_stride: per clique-search item, its best key and valid count
    int32_t rec_stride;       // 2 x the most clique-search items of a pair (k1_cap)
    int32_t pool_cap;
    int32_t *pivots_plain;    // max_batch x pool_cap x 3
    int32_t *pivots;          // pivots the clique search uses: max_batch x piv_stride x 3
    int32_t piv_stride;       // pool_cap in plain mode (pivots == pivots_plain), k1_cap in learned mode
    int32_t *cliques;         // max_batch x h_cap x 3
    float *poses;             // max_batch x h_cap x 12
    int32_t *inl;             // max_batch x h_cap
    float *gscore;            // max_batch x h_cap error-based scores (metric != 0)
    int32_t metric;           // hypothesis ranking: 0 inlier number, 1 MAE form, 2 MSE form
    int32_t h_cap;
    int32_t *rowstat;         // max_batch x max_n x 20 feature accumulators (learned mode): degree, two unused, 16 bins, one unused
    // row sums and maxima of the SC2 matrix in parts that the SC2 kernels store (learned mode), with segmax: row i's
    // sum over the pairs i < j of each 64-column segment (as segmax), and per 128-row block and column the sum and
    // maximum over the pairs i < j of the block (npad x npad / 128 from g_off / 128)
    int32_t *rowsum, *colsum;
    uint16_t *colmax;
    int32_t *mark;            // max_batch x max_n: row claimed by a candidate-feature workgroup
    int32_t feat_all;         // learned features for every match (training) instead of the pool's
    uint16_t *feat;           // max_batch x max_n x 19 bfloat16 features
    float *scores;            // max_batch x max_n learned scores
    tr_result *out;
    uint8_t *masks;           // nullable; pair b's mask starts at pairs[b].pt_off
    int32_t learned;          // learned pivot mode / feature accumulation on
    int32_t rank_in_hyp;      // learned pool of at most kFusedPool entries: the hypothesis kernel orders it
    // Profiled calls only (null otherwise): the hypothesis kernel's phase durations in ticks of
    // the 100 MHz real-time clock, per work item (max_batch x rec_stride / 2 x 4: clique search,
    // rigid fits, scoring, records), and their sums over calls (kProfSlots counters).
    uint32_t *hyp_prof;
    unsigned long long *prof_acc;
};

// Sums of the hypothesis kernel's phases over profiled calls (prof_acc slots).
enum { kProfSearch = 0, kProfFit, kProfScore, kProfRecords, kProfSelect, kProfItems, kProfPairs, kProfSlots };

// Length of a difference vector in float32: first square rounded, the other
// two fused, then the correctly rounded square root (the order is part of the
// bit-exact contract of C).
__device__ __forceinline__ float length32(float ax, float ay, float az)
{
    float s = ax * ax;
    s = __builtin_fmaf(ay, ay, s);
    s = __builtin_fmaf(az, az, s);
    return __builtin_sqrtf(s);
}

// Learned reorder key of plain pool entry r (smaller = earlier): e = s_i + s_j descending, then
// the plain rank r; keys are distinct. fb: the pair's scores are not all finite, keep plain order.
__device__ __forceinline__ uint64_t reorder_key(const int32_t *pl, const float *sc, int r, bool fb)
{
    uint32_t hi = 0;
    if (!fb) {
        const float e = (sc[pl[3 * r]] + sc[pl[3 * r + 1]]) + 0.0f;   // +0.0f folds -0 into +0
        const uint32_t u = __float_as_uint(e);
        const uint32_t ord = (u & 0x80000000u) ? ~u : (u | 0x80000000u);   // ascending float order
        hi = ~ord;                                                            // descending
    }
    return ((uint64_t)hi << 32) | (uint32_t)r;
}

// Number of the keys in [q0, q1) (LDS, padded with ~0 to a multiple of 16) smaller than `mine`,
// eight 16-byte broadcast reads in flight; q0, q1 multiples of 16.
__device__ __forceinline__ int count_smaller(const uint64_t *keys, int q0, int q1, uint64_t mine)
{
    int rk = 0;
    for (int q = q0; q < q1; q += 16) {
        uint4 a[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = *reinterpret_cast<const uint4 *>(&keys[q + 2 * u]);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            rk += (((uint64_t)a[u].y << 32) | a[u].x) < mine;
            rk += (((uint64_t)a[u].w << 32) | a[u].z) < mine;
        }
    }
    return rk;
}

// Largest b in [0, B) with pre[b] <= item (pre is non-decreasing, pre[0] = 0).
__device__ __forceinline__ int find_pair(const int32_t *pre, int B, int item)
{
    int lo = 0, hi = B - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= item) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Per-pair sizes of a valid pair (3 <= n <= max_n): the descriptor and the
// work items of every stage. The device planner and single-pair calls (which
// compute their plan in registers) use the same formulas.
__host__ __device__ inline PairDesc pair_desc_of(int32_t n, int32_t pt_off, int64_t arena_off, int32_t pool)
{
    PairDesc d;
    d.n = n;
    d.npad = (n + kSc2Tile - 1) / kSc2Tile * kSc2Tile;
    d.pt_off = pt_off;
    const int64_t pairs_all = (int64_t)n * (n - 1) / 2;
    d.kpiv = (int32_t)(pairs_all < pool ? pairs_all : pool);
    d.c_off = arena_off;
    d.g_off = arena_off;
    return d;
}

// Place of row (column) x's k-th of `parts` partial values: 32 rows together, so that a kernel stores whole lines and
// one that sums a row's parts stays within few pages.
__host__ __device__ inline int32_t part_at(int32_t x, int32_t k, int32_t parts)
{
    return ((x >> 5) * parts + k) * 32 + (x & 31);
}

// Byte offset, from a lane's piece of the first two 128-column blocks of C, of step s of the dense SC2 product
// (two blocks, 2 x kbs bytes, a step; ns steps). The loop asks for up to two steps past the last: these read the
// last one's blocks again (unused), so that no load leaves the pair's bits.
__host__ __device__ inline int32_t sc2_step_offset(int32_t s, int32_t ns, uint32_t kbs)
{
    return (s < ns ? s : ns - 1) * (int32_t)(2 * kbs);
}

// Segments (64 columns) of 64 rows that a wave of the row scan takes: sixteen, whose maxima it reads at once; one
// in small pairs, which would fill few waves. Up to 512 matches the four waves of a workgroup share one segment by
// rows (n = 300: 5.9 us, 6.2 apart); beyond, the workgroups' atomics cost more than that saves (n = 1000: 8.4 us,
// 5.9 apart).
__host__ __device__ inline int32_t collect_segs(int32_t n)
{
    return n <= 1024 ? 1 : 16;
}

__host__ __device__ inline bool collect_shared(int32_t n)
{
    return n <= 512;
}

__host__ __device__ inline int64_t stage_items(int stage, int32_t n, int32_t H, int32_t sp)
{
    const int64_t npad = (n + kSc2Tile - 1) / kSc2Tile * kSc2Tile;
    const int64_t nbc = npad / kCompatTile, nbs = npad / kSc2Tile;
    switch (stage) {
    case kPrep: return (n + kPrepRows - 1) / kPrepRows;
    case kCompat: return nbc * (nbc + 1) / 2;
    case kSc2: return nbs * (nbs + 1) / 2;
    case kSp: { const int64_t nb = sp > 0 ? (n + sp - 1) / sp : 0; return nb * (nb + 1) / 2; }   // bit-count tiles of edge sp
    case kCollect: {
        const int64_t nb = (n + 63) / 64, sg = collect_segs(n), units = nb * ((nb + sg - 1) / sg);
        return collect_shared(n) ? units : (units + 3) / 4;
    }
    case kRowBlk: return (n + kRowsPerItem - 1) / kRowsPerItem;
    default: return (int64_t)((H + kScoreHyp - 1) / kScoreHyp) * ((n + kScorePts - 1) / kScorePts);
    }
}

// Pivots per work item of the hypothesis kernel: ppw, less while an item would still make more than one pass of eight
// poses over the matches and the smaller items all run at once on the `slots` workgroups that the CUs hold (one of eight
// waves each; two of four for the error rankings). One item more per CU costs a whole second round: whole calls (us) with
// items in one round / halved again, past it: K1 = 1000, K2 = 8 on N = 300 53.0 / 62.8, on 2749 77.6 / 87.7, on 6000
// 123.4 / 135.6, 100 pairs of 100 matches, K1 = 32 86.5 / 93.7. Items left larger than that / halved: N = 2749,
// K1 = 250, K2 = 8 (63 items of 4 pivots, 250 of one) 53 / 32 us of the kernel; MAE ranking, K1 = 550 on N = 2749 (138
// items of 4, 275 of two) 103.1 / 86.7.
__host__ __device__ inline int32_t hyp_item_pivots(int32_t B, int32_t k1, int32_t k2, int32_t ppw, int32_t slots)
{
    while (ppw > 1 && ppw * k2 > 8 && (int64_t)B * ((k1 + ppw / 2 - 1) / (ppw / 2)) <= slots) ppw /= 2;
    return ppw;
}

// Rows per work item (one wave) of the compatibility kernel, for a list of `tiles` tiles: long items
// amortise the item's loads and transposes, short ones spread a short list over the CUs.
// Measured at 8 / 16 / 32 / 64 / 128 rows (us): N = 300 6.1 / 6.8 / 9.4, N = 1000 6.0 / 7.3 / 9.8,
// N = 2749 (253 tiles) 9.1 / 9.0 / 10.8, N = 5000 (820) 20.5 / 18.3 / 17.2 / 19.7 / 29.7, N = 20000 (12403)
// 199 / 143 / 116 / 112 / 107, 256 pairs 1580 / 1091 / 856 / 800 / 750. (With 64 x 64 tiles per workgroup, two
// square roots a pair and packing through LDS: 6.1, 6.8, 10.6, 22.6, 229 and 2060.)
__host__ __device__ inline int32_t compat_rows(int64_t tiles, int32_t num_cus)
{
    return tiles <= num_cus ? 8 : tiles <= 2 * num_cus ? 16 : tiles <= 16 * num_cus ? 32 : 128;
}

// Tile edge of the SC2 bit-count kernel, by the number of tiles of each edge 256, 512, 768 and 1024 over all pairs:
// larger tiles read each row's bits fewer times, smaller ones spread a short list over the CUs (one workgroup each).
// The cost of a round of tiles is its edges, plus what a tile costs besides (as much as 2^17 entries). 0: no tiles, a
// list that one round of 256-tiles holds takes the product, whatever limit is asked for. Bit counts / product there
// (us a call, 1.5 % edges): one pair of 1000 106 / 74, of 3000 113 / 86, of 5000 130 / 111, sixteen of 1000 183 / 147;
// beyond it one of 8000 176 / 190, sixteen of 3000 309 / 285, of 5000 568 / 629.
constexpr int kSpEdges = 4;
__host__ __device__ inline int32_t sparse_tile(const int32_t *tiles, int32_t num_cus)
{
    if (tiles[0] <= num_cus) return 0;
    int32_t best = 0;
    int64_t cost = INT64_MAX;
    for (int k = kSpEdges; k >= 1; --k) {
        const int64_t rounds = (tiles[k - 1] + num_cus - 1) / num_cus, c = rounds * (65536 * k * k + (1 << 17));
        if (c < cost) {
            cost = c;
            best = 256 * k;
        }
    }
    return best;
}

// Work lists: all items of a stage, pair after pair, in the plan's slot order: for batches of
// 16 pairs or more, the pairs sorted by decreasing size (npad; pairs of one size in index order) and dealt to the eight XCDs, each
// XCD's pairs in size order, so that eight SC2 ranges of equal cost hold like mixes of sizes and
// a workgroup striding through a list takes costly items first. A single-pair call (n1 > 0)
// derives everything from n1; a batch reads the device plan.
__device__ __forceinline__ int stage_total(const Work &w, int stage)
{
    return w.n1 ? (int)stage_items(stage, w.n1, w.H, w.sp_tile) : w.plan->total[stage];
}

__device__ __forceinline__ int sc2_sparse_edge(const Work &w)
{
    return w.n1 ? w.sp_tile : w.plan->sp_tile;
}

__device__ __forceinline__ int compat_item_rows(const Work &w)
{
    return w.n1 ? w.compat_rows : w.plan->compat_rows;
}

// The pair in slot k of the cost order (kernels with one workgroup, or a fixed number, per
// pair take their pairs in this order too).
__device__ __forceinline__ int batch_pair(const Work &w, int k)
{
    return w.n1 ? k : w.pre[kOrderRow * w.pre_stride + k];
}

// The pair an item belongs to, and the item's index inside that pair.
__device__ __forceinline__ int stage_pair(const Work &w, int stage, int item, int &local)
{
    if (w.n1) {
        local = item;
        return 0;
    }
    const int32_t *pre = w.pre + stage * w.pre_stride;
    const int k = find_pair(pre, w.plan->B, item);
    local = item - pre[k];
    return w.pre[kOrderRow * w.pre_stride + k];
}

// The same lookup from a copy in LDS of a stage's prefix sums and the slot order, for kernels
// with many short items (the binary search then takes no device-memory round trips). Batches of
// at most kSlotCacheMax pairs; the copy is made by slot_cache_fill, followed by a barrier.
constexpr int kSlotCacheMax = 1024;
struct SlotCache {
    int32_t pre[kSlotCacheMax + 1];
    int32_t order[kSlotCacheMax];
};

__device__ __forceinline__ bool slot_cache_fill(const Work &w, int stage, SlotCache &c)
{
    if (w.n1 || w.plan->B > kSlotCacheMax) return false;
    const int B = w.plan->B;
    for (int k = threadIdx.x; k <= B; k += blockDim.x) {
        c.pre[k] = w.pre[stage * w.pre_stride + k];
        if (k < B) c.order[k] = w.pre[kOrderRow * w.pre_stride + k];
    }
    return true;
}

__device__ __forceinline__ int stage_pair_cached(const Work &w, int stage, const SlotCache &c, bool cached, int item,
                                                 int &local)
{
    if (!cached) return stage_pair(w, stage, item, local);
    const int k = find_pair(c.pre, w.plan->B, item);
    local = item - c.pre[k];
    return c.order[k];
}

// First item of pair b in a stage's list, and its item count.
__device__ __forceinline__ int stage_first(const Work &w, int stage, int b)
{
    return w.n1 ? 0 : w.pre[stage * w.pre_stride + w.pre[kSlotRow * w.pre_stride + b]];
}

__device__ __forceinline__ int stage_count(const Work &w, int stage, int b)
{
    if (w.n1) return (int)stage_items(stage, w.n1, w.H, w.sp_tile);
    const int k = w.pre[kSlotRow * w.pre_stride + b];
    return w.pre[stage * w.pre_stride + k + 1] - w.pre[stage * w.pre_stride + k];
}

__device__ __forceinline__ PairDesc pair_desc(const Work &w, int b)
{
    return w.n1 ? pair_desc_of(w.n1, 0, 0, w.pool) : w.pairs[b];
}

// ---- launchers (one per kernel family); each returns the launch's hipError_t ----
hipError_t launch_plan(const Work &w, const int32_t *offsets, int32_t n_single, int32_t B,
                       int32_t max_n, int num_cus, PairDesc *pairs, PairState *state, Plan *plan, int32_t *pre,
                       hipStream_t s);
hipError_t launch_compat(const Work &w, int64_t tiles, int cap, hipStream_t s);
hipError_t launch_compat_features(const Work &w, int64_t items, int cap, hipStream_t s);
hipError_t launch_sc2_sparse(const Work &w, int64_t tiles, int num_cus, hipStream_t s);
hipError_t launch_sc2(const Work &w, int64_t items, int num_cus, hipStream_t s);
hipError_t launch_pivots(const Work &w, int B, int grid_rows, int num_cus, hipStream_t s);
hipError_t launch_hyp(const Work &w, int B, int ppw, int grid, int num_cus, hipStream_t s);
hipError_t launch_fit_triplets(const float *src, const float *dst, int n, const int32_t *tri, int T, float *poses,
                               int32_t *ok, int grid, hipStream_t s);
hipError_t launch_score_poses(const float *src, const float *dst, int n, const float *poses, int P, float theta,
                              int metric, int32_t *in_out, float *score_out, int num_cus, hipStream_t s);
hipError_t setup_hyp_kernels();

// Once per process and device, before any launch (and so outside stream capture):
// raise the dynamic-LDS limits of the kernels that need more than 64 KiB.
hipError_t setup_graph_kernels();
hipError_t setup_pivot_kernels();

}  // namespace tr
