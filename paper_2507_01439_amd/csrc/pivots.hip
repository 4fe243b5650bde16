// Pivot selection (Eq. 4) on gfx950.
//
// The pivots are the first K pairs i < j of the O2Graph ordered by
// (weight desc, i asc, j asc), K = min(K1, N(N-1)/2). Weights are integers
// below N, so the K-th largest weight alpha comes from an exact histogram.
// Every pair heavier than alpha is a pivot, and the first m pairs of weight
// alpha in row-major order fill the remaining slots.
//
//   (the SC2 kernels leave kHistGroups weight histograms per pair and the
//   maximum of each row's 64-column segments of the upper triangle)
//   k_thresh   sums the histograms; finds alpha, the pairs heavier than it
//              (c_gt) and the ties to take (m); sums the compatibility
//              kernel's per-tile counts (boundary pairs, edges, non-finite);
//              small single pairs do this at the start of k_rowscan
//   k_rowscan  collects every pair of weight >= alpha when they fit the pool
//              (fast path), else the pairs heavier than alpha and, per row and
//              per row block, the count of pairs of weight alpha (ordered path)
//   k_sort     ranks the collected keys by (w desc, i asc, j asc) and keeps
//              the first K; on the ordered path it places the first m ties in
//              row-major order after the c_gt heavier pairs
// The key set is exact on both paths and every position is decided by a rank
// or a row-major tie index, so the pivot list does not depend on the order
// atomics were served in.
#include "common.h"

#include <algorithm>
#include <type_traits>

namespace tr {
namespace {

// Inclusive prefix sum over the 64 lanes: shifts by 1, 2, 4, 8 inside each
// 16-lane row, then the last lane of row 0 is added to row 1 and of row 2 to
// row 3, then lane 31 to rows 2 and 3 (DPP row_shr / row_bcast, no LDS).
__device__ __forceinline__ int wave_incl_scan(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1, 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2, 3
    return x;
}

template <typename T>
__device__ T block_exclusive_scan(T v, T *lds, T &total)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    T x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        T y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) lds[wid] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        T acc = 0;
        for (int k = 0; k < nw; ++k) { T t = lds[k]; lds[k] = acc; acc += t; }
        lds[nw] = acc;
    }
    __syncthreads();
    T res = lds[wid] + x - v;
    total = lds[nw];
    __syncthreads();
    return res;
}

// Sort key: smaller key = earlier pivot.
__device__ __forceinline__ uint64_t pivot_key(uint32_t w, uint32_t i, uint32_t j)
{
    return ((uint64_t)(0xFFFFu - w) << 40) | ((uint64_t)i << 20) | (uint64_t)j;
}

constexpr int kMaxFirst = 2048;

struct Threshold {
    int32_t alpha, c_gt, m_eq, fast, ncand;   // as in PairState
};

// alpha = the K-th largest weight over all N(N-1)/2 pairs (zeros included), by a workgroup of NT threads.
// hs: n ints of LDS.
template <int NT>
__device__ Threshold pair_threshold(const Work &w, const PairDesc &d, int b, int32_t *hs)
{
    __shared__ int32_t wtot[NT / 64];
    __shared__ Threshold res;
    const int64_t K = d.kpiv;
    const int tid = threadIdx.x;
    const int32_t *gh = w.ghist + (int64_t)b * kHistGroups * w.hist_stride;
    // bin 0 of each copy holds the largest weight it saw: bins past that are empty. Worth its round trip where the
    // copies take long to read (us:
    // k_thresh at N = 20000 24.3 -> 7.5, the fused scan at N = 5000 11.2 -> 8.5, at 2749 9.5 -> 8.1; at 1000 7.6 -> 8.0)
    int n = d.n;
    if (n > kMaxFirst) {
        int top = 0;
#pragma unroll
        for (int g = 0; g < kHistGroups; ++g) top = max(top, gh[(int64_t)g * w.hist_stride]);
        n = min(n, top + 1);
    }
    // eight consecutive bins per thread: two 16-byte loads from each copy, all issued before any is
    // summed (the pass is latency-bound: 1024 threads take one round up to 8192 bins); bins at or past n are
    // empty or never written and are not summed (the copies are padded to a multiple of 8)
    for (int v0 = 8 * tid; v0 < n; v0 += 8 * NT) {
        int4 c[kHistGroups][2];
#pragma unroll
        for (int g = 0; g < kHistGroups; ++g) {
            c[g][0] = *reinterpret_cast<const int4 *>(gh + (int64_t)g * w.hist_stride + v0);
            c[g][1] = *reinterpret_cast<const int4 *>(gh + (int64_t)g * w.hist_stride + v0 + 4);
        }
        int32_t sum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int g = 0; g < kHistGroups; ++g) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                sum[4 * h] += c[g][h].x;
                sum[4 * h + 1] += c[g][h].y;
                sum[4 * h + 2] += c[g][h].z;
                sum[4 * h + 3] += c[g][h].w;
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (v0 + u < n) hs[v0 + u] = sum[u];
    }
    __syncthreads();
    // bins w = 1 .. n-1 walked from the top: thread t sums the contiguous positions u0 .. u1-1
    // (u = n-1-w); an in-wave scan and the wave totals give each thread the count above
    // its range, and the thread whose range holds the K-th largest weight walks it (counts stay
    // below n(n-1)/2 < 2^31)
    const int nb = max(n - 1, 0);
    const int cs = (nb + NT - 1) / NT;
    const int u0 = min(nb, tid * cs), u1 = min(nb, u0 + cs);
    int local = 0;
    for (int u = u0; u < u1; ++u) local += hs[n - 1 - u];
    const int incl = wave_incl_scan(local);
    if ((tid & 63) == 63) wtot[tid >> 6] = incl;
    __syncthreads();
    int64_t tot = 0, before = 0;
#pragma unroll
    for (int v = 0; v < NT / 64; ++v) {
        const int t = wtot[v];
        before += v < (tid >> 6) ? t : 0;
        tot += t;
    }
    const int64_t excl = before + incl - local;
    // pairs of weight alpha: the histogram bin, or every pair of weight 0
    auto found = [&](int alpha, int64_t above, int64_t ties) {
        const bool fast = above + ties <= w.pool_cap;
        res = Threshold{alpha, (int32_t)above, (int32_t)(K - above), fast, fast ? (int32_t)(above + ties) : (int32_t)K};
    };
    if (tid == 0 && K > tot) found(0, tot, (int64_t)d.n * (d.n - 1) / 2 - tot);
    if (K <= tot && excl < K && K <= excl + local) {
        int64_t cum = excl;
        for (int u = u0; u < u1; ++u) {
            const int wt = n - 1 - u;
            const int64_t c = hs[wt];
            if (cum + c >= K) {
                found(wt, cum, c);
                break;
            }
            cum += c;
        }
    }
    __syncthreads();
    return res;
}

__device__ __forceinline__ void store_threshold(PairState &st, const Threshold &t)
{
    st.alpha = t.alpha;
    st.c_gt = t.c_gt;
    st.m_eq = t.m_eq;
    st.fast = t.fast;
    st.ncand = t.ncand;
}

// Boundary pairs, edges and non-finite input of the pair, summed over its compatibility items by NT threads; the
// first eight items per thread are loaded at construction.
template <int NT>
struct Tally {
    static constexpr int kItems = 8;
    int t0, t1;
    uint32_t tv[kItems];

    __device__ __forceinline__ void load(const Work &w, int tb)
    {
#pragma unroll
        for (int u = 0; u < kItems; ++u) {
            const int t = tb + NT * u;
            tv[u] = t < t1 ? w.cnt_part[t] : 0;
        }
    }

    __device__ __forceinline__ Tally(const Work &w, int b)
    {
        const int per = kCompatTile / compat_item_rows(w);   // work items per list tile
        t0 = per * stage_first(w, kCompat, b);
        t1 = t0 + per * stage_count(w, kCompat, b);
        load(w, t0 + (int)threadIdx.x);
    }

    __device__ void store(const Work &w, int b)
    {
        __shared__ int32_t tally[NT / 64][3];
        int cc[3] = {0, 0, 0};
        for (int tb = t0 + (int)threadIdx.x;;) {
#pragma unroll
            for (int u = 0; u < kItems; ++u) {
                cc[0] += (tv[u] >> 15) & 0x7FFFu;
                cc[1] += tv[u] & 0x7FFFu;
                cc[2] |= tv[u] >> 30;
            }
            tb += NT * kItems;
            if (tb >= t1) break;
            load(w, tb);
        }
#pragma unroll
        for (int f = 0; f < 3; ++f) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) cc[f] += __shfl_xor(cc[f], o, 64);
        }
        if ((threadIdx.x & 63) == 0) {
            tally[threadIdx.x >> 6][0] = cc[0];
            tally[threadIdx.x >> 6][1] = cc[1];
            tally[threadIdx.x >> 6][2] = cc[2];
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int tb = 0, te = 0, tn = 0;
            for (int v = 0; v < NT / 64; ++v) {
                tb += tally[v][0];
                te += tally[v][1];
                tn |= tally[v][2];
            }
            w.state[b].n_boundary = tb;
            w.state[b].n_edges = te;
            w.state[b].nonfinite = tn != 0;
        }
    }
};

__global__ void __launch_bounds__(1024) k_thresh(Work w)
{
    extern __shared__ int32_t hs[];
    const int b = batch_pair(w, blockIdx.x);
    const PairDesc d = pair_desc(w, b);
    // this call's counters of the pair (collection regions, clique-search tickets) start at zero;
    // the later kernels of the call update them
    for (int k = threadIdx.x; k < w.tick_stride / kTickLine; k += 1024) w.tick[(int64_t)b * w.tick_stride + k * kTickLine] = 0;
    if (d.kpiv <= 0) return;
    Tally<1024> tally(w, b);
    const Threshold t = pair_threshold<1024>(w, d, b, hs);
    if (threadIdx.x == 0) store_threshold(w.state[b], t);
    tally.store(w, b);
}

// ---------------------------------------------------------------- row scan

constexpr int kFuseThreshMax = 8192;   // matches of a single pair up to which the row scan finds the threshold itself
constexpr int kCollectCap = 1024;   // keys a workgroup stages in LDS before its one global reservation

// The pairs that can be pivots, appended to the workgroup's XCD region of the pool in no particular order (the
// rank sort fixes it). A workgroup stages its keys in LDS, reserves its range with one atomic and copies them
// out; if an item holds more than kCollectCap keys it reserves the count first and writes straight to the pool
// on a second read.
//
// Fast path (every pair of weight >= alpha fits the pool): a wave takes 64 rows by 16 segments of 64 columns,
// reads the segments' maxima (a row per lane) and then only the segments that reach alpha, eight lanes each.
// There are at most as many as collected keys, so the pass costs its round trips: of the weights, which a
// whole-row scan mostly read (rows nearly all hold some pivot), a few per cent are touched.
// 256 pairs of 800 to 5000 matches 440 -> 72 us, N = 20000 29 -> 10.3, N = 5000 8.9 -> 6.5; N = 300 5.4 -> 5.9 (from
// one row per wave, read whole where its maximum reaches alpha).
//
// Ordered path: the pairs heavier than alpha (there are c_gt < K of them), one row per wave, all of its 16-byte
// chunks loaded before any is used; rows whose maximum is below alpha are not read. Each chunk gives two 8-bit
// masks: the pairs (inside i < j < n) heavier than alpha and those equal to it. Besides: per row, the pairs of
// weight alpha and a mask of the 512-column segments holding any; per row block, their sum. The sort kernel
// locates the first m ties in row-major order from these.
//
// FUSED (a single pair of few matches): every workgroup finds the threshold itself, from the same histograms, in
// place of a kernel before this one; the first stores it, the last sums the pair's counts. No more workgroups than
// CUs, as each reads all copies of the histogram. Both kernels / this one alone (us, without the gap between them):
// N = 300 11.3 / 7.4, N = 1000 11.3 / 7.6, N = 2749 12.1 / 8.1, N = 5000 13.9 / 8.5; whole calls of 5000 matches
// 87.9 / 84.1, of 8000 169.2 / 164.7, of 10000 264.4 / 262.8, of 13000 468.6 / 472.1.
template <bool FUSED>
__global__ void __launch_bounds__(256) k_rowscan(Work w)
{
    extern __shared__ int32_t hs[];   // FUSED
    __shared__ uint64_t buf[kCollectCap];
    __shared__ int32_t nbuf, base;
    __shared__ int32_t part[4];
    __shared__ uint16_t list[4][64 * 16];
    __shared__ SlotCache slots;
    // batches of up to kInfoMax pairs: each slot's threshold, path and sizes in LDS as well, so an
    // item starts with no device-memory round trip but its segments' maxima
    constexpr int kInfoMax = 256;
    struct SlotInfo {
        int32_t alpha, fast, kpiv, n, npad, pad;
        int64_t g_off;
    };
    __shared__ SlotInfo info[kInfoMax];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // the pool region and counter of this workgroup's XCD (workgroup g runs on XCD g mod 8)
    const int rgn = blockIdx.x & (kCollectRegions - 1);
    Threshold own{};
    if (FUSED) {
        const PairDesc d = pair_desc(w, 0);
        if (d.kpiv <= 0) return;
        if (blockIdx.x == gridDim.x - 1) Tally<256>(w, 0).store(w, 0);
        own = pair_threshold<256>(w, d, 0, hs);
        if (blockIdx.x == 0 && tid == 0) store_threshold(w.state[0], own);
    }
    const bool cached = !FUSED && slot_cache_fill(w, kCollect, slots);
    const bool with_info = cached && w.plan->B <= kInfoMax;
    __syncthreads();
    // some pair takes the ordered path (may, where the pairs are not all known here)
    bool slow = !with_info;
    if (with_info)
        for (int k = tid; k < w.plan->B; k += blockDim.x) {
            const int b = slots.order[k];
            const PairState st = w.state[b];
            const PairDesc d = w.pairs[b];
            info[k] = SlotInfo{st.alpha, st.fast, d.kpiv, d.n, d.npad, 0, d.g_off};
            slow |= d.kpiv > 0 && !st.fast;
        }
    if (with_info) slow = __syncthreads_or(slow);
    // an item's pair, path and place in the pair; false: nothing to do (the same for the whole workgroup)
    auto open_item = [&](Stage stage, int item, bool ordered, int &blk, int &b, int &alpha, PairDesc &d) {
        int fast;
        if (with_info) {
            const int k = find_pair(slots.pre, w.plan->B, item);
            blk = item - slots.pre[k];
            b = slots.order[k];
            const SlotInfo &f = info[k];
            alpha = f.alpha;
            fast = f.fast;
            d.kpiv = f.kpiv;
            d.n = f.n;
            d.npad = f.npad;
            d.g_off = f.g_off;
        } else {
            b = stage_pair_cached(w, stage, slots, cached, item, blk);
            d = pair_desc(w, b);
            alpha = FUSED ? own.alpha : w.state[b].alpha;
            fast = FUSED ? own.fast : w.state[b].fast;
        }
        return d.kpiv > 0 && ordered == !fast;
    };
    // stage (direct = false) or write (direct = true, at base + ...) the keys of the set bits of hits[v]: pairs
    // (i[v], 8 c[v] + e) with the weights q[v]
    auto append = [&](auto n_c, const uint32_t *hits, const int *i, const int *c, const uint4 *q, bool direct, uint64_t *cand) {
        constexpr int N = decltype(n_c)::value;
        int m = 0;
#pragma unroll
        for (int v = 0; v < N; ++v) m += __builtin_popcount(hits[v]);
        const int incl = wave_incl_scan(m);
        const int tot = __builtin_amdgcn_readlane(incl, 63);
        int off = 0;
        if (lane == 63) off = atomicAdd(&nbuf, tot);
        off = __builtin_amdgcn_readlane(off, 63) + incl - m;
#pragma unroll
        for (int v = 0; v < N; ++v) {
            const uint32_t uw[4] = {q[v].x, q[v].y, q[v].z, q[v].w};
            for (uint32_t h = hits[v]; h; h &= h - 1) {
                const int e = __builtin_ctz(h);
                const uint32_t lo = e & 2 ? uw[1] : uw[0], hi = e & 2 ? uw[3] : uw[2], x = e & 4 ? hi : lo;
                const uint64_t key = pivot_key(e & 1 ? x >> 16 : x & 0xFFFFu, i[v], 8 * c[v] + e);
                if (direct) {
                    if (base + off < w.pool_cap) cand[base + off] = key;
                } else if (off < kCollectCap) {
                    buf[off] = key;
                }
                ++off;
            }
        }
    };
    // the item's keys into the pool: `scan` stages them, or writes them if the stage is too small
    auto collect = [&](int b, uint64_t *cand, auto &&scan) {
        if (tid == 0) nbuf = 0;
        __syncthreads();
        scan(false);
        __syncthreads();
        const int n_wg = nbuf;
        __syncthreads();   // every thread has read nbuf before it is reset
        if (n_wg > 0) {
            if (tid == 0) base = atomicAdd(&w.tick[(int64_t)b * w.tick_stride + rgn * kTickLine], n_wg);
            __syncthreads();
            if (n_wg <= kCollectCap) {
                for (int k = tid; k < n_wg; k += 256)
                    if (base + k < w.pool_cap) cand[base + k] = buf[k];
            } else {
                if (tid == 0) nbuf = 0;
                __syncthreads();
                scan(true);
            }
        }
    };
    // ---- fast path
    const int units = stage_total(w, kCollect);
    for (int item = blockIdx.x; item < units; item += gridDim.x) {
        int blk, b, alpha;
        PairDesc d;
        if (!open_item(kCollect, item, false, blk, b, alpha, d)) continue;
        const int nseg = (d.n + 63) / 64, segs = collect_segs(d.n), u = collect_shared(d.n) ? blk : 4 * blk + wv, rb = u % nseg, s0 = u / nseg * segs;
        uint64_t *cand = w.cand + ((int64_t)b * kCollectRegions + rgn) * w.pool_cap;
        const uint16_t *G = w.G + d.g_off + (int64_t)(64 * rb) * d.npad;
        int nh = 0;   // the wave's segments that reach alpha: row | segment << 6 in `list`
        if (s0 < nseg && s0 + segs > rb) {   // segments left of the rows' own hold no pair
            const int i = !collect_shared(d.n) || lane >> 4 == wv ? 64 * rb + lane : d.n;   // n: not this wave's row
            const uint16_t *sm = w.segmax + d.g_off / 64 + part_at(64 * rb + lane, 0, d.npad / 64);
            int m[16];
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const int s = s0 + t;
                m[t] = t < segs && s >= rb && s < nseg && i < d.n ? (int)sm[32 * s] : -1;
            }
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const bool hit = m[t] >= alpha;
                const uint64_t mask = __ballot(hit);
                if (hit)
                    list[wv][nh + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0))] =
                        (uint16_t)(lane | t << 6);
                nh += __builtin_popcountll(mask);
            }
        }
        collect(b, cand, [&](bool direct) {
            for (int h0 = 0; h0 < nh; h0 += 64) {
                uint4 q[8];
                int row[8], c[8];
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    const int h = h0 + 8 * v + (lane >> 3), x = list[wv][min(h, nh - 1)];
                    row[v] = h < nh ? x & 63 : -1;
                    c[v] = 8 * (s0 + (x >> 6)) + (lane & 7);
                    q[v] = *reinterpret_cast<const uint4 *>(G + (int64_t)(x & 63) * d.npad + 8 * c[v]);
                }
                uint32_t hits[8];
                bool any = false;
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    // bit e: pair (i, 8c + e) lies in i < j < n and weighs at least alpha
                    const int i = 64 * rb + row[v];
                    const int lo = min(max(i + 1 - 8 * c[v], 0), 8), hi = min(max(d.n - 8 * c[v], 0), 8);
                    const uint32_t range = row[v] < 0 ? 0u : ((1u << hi) - 1u) & ~((1u << lo) - 1u);
                    const uint32_t uw[4] = {q[v].x, q[v].y, q[v].z, q[v].w};
                    hits[v] = 0;
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        hits[v] |= ((uint32_t)((int)(uw[k] & 0xFFFFu) >= alpha) << (2 * k)) |
                                   ((uint32_t)((int)(uw[k] >> 16) >= alpha) << (2 * k + 1));
                    hits[v] &= range;
                    any |= hits[v] != 0;
                    row[v] = i;
                }
                if (__any(any)) append(std::integral_constant<int, 8>(), hits, row, c, q, direct, cand);
            }
        });
        __syncthreads();   // buf, nbuf, base and list are the next item's
    }
    if (FUSED ? own.fast != 0 : w.n1 ? w.state[0].fast != 0 : !slow) return;
    // ---- ordered path
    __syncthreads();
    if (!FUSED) slot_cache_fill(w, kRowBlk, slots);
    __syncthreads();
    const int total = stage_total(w, kRowBlk);
    for (int item = blockIdx.x; item < total; item += gridDim.x) {
        int blk, b, alpha;
        PairDesc d;
        if (!open_item(kRowBlk, item, true, blk, b, alpha, d)) continue;
        const int c1 = (d.n + 7) >> 3;
        const int i = blk * kRowsPerItem + wv;
        bool live = i < d.n && alpha <= 0;
        if (i < d.n && alpha > 0) {   // some segment reaches alpha
            const uint16_t *sm = w.segmax + d.g_off / 64 + part_at(i, 0, d.npad / 64);
            for (int s = (i >> 6) + lane; s < (d.n + 63) / 64; s += 64) live |= (int)sm[32 * s] >= alpha;
            live = __any(live);
        }
        const uint16_t *row = w.G + d.g_off + (int64_t)i * d.npad;
        const int c_lo = (i + 1) >> 3;
        uint64_t *cand = w.cand + ((int64_t)b * kCollectRegions + rgn) * w.pool_cap;
        // ties / segs: the lane's pairs of weight alpha and the segments holding any
        int ties = 0;
        uint64_t segs = 0;
        collect(b, cand, [&](bool direct) {
            if (!live) return;
            for (int c0 = c_lo; c0 < c1; c0 += 1024) {
                uint4 q[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    const int c = c0 + 64 * u + lane;
                    q[u] = c < c1 ? *reinterpret_cast<const uint4 *>(row + 8 * c) : make_uint4(0, 0, 0, 0);
                }
                const int steps = min(16, (c1 - c0 + 63) >> 6);   // the same on every lane
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    if (u >= steps) continue;   // uniform: the loop stays unrolled
                    const int c = c0 + 64 * u + lane;
                    // bit e: pair (i, 8c + e) lies in i < j < n and weighs more than / exactly alpha
                    const int lo = min(max(i + 1 - 8 * c, 0), 8), hi = min(max(d.n - 8 * c, 0), 8);
                    const uint32_t range = ((1u << hi) - 1u) & ~((1u << lo) - 1u);
                    const uint32_t uw[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
                    uint32_t hge = 0, heq = 0;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        hge |= ((uint32_t)((int)(uw[k] & 0xFFFFu) >= alpha) << (2 * k)) |
                               ((uint32_t)((int)(uw[k] >> 16) >= alpha) << (2 * k + 1));
                        heq |= ((uint32_t)((int)(uw[k] & 0xFFFFu) == alpha) << (2 * k)) |
                               ((uint32_t)((int)(uw[k] >> 16) == alpha) << (2 * k + 1));
                    }
                    heq &= range;
                    if (!direct) {
                        ties += __builtin_popcount(heq);
                        if (__any(heq != 0)) segs |= 1ull << ((c0 - c_lo) / 64 + u);   // at most 64 segments (N < 32768)
                    }
                    const uint32_t hits = hge & range & ~heq;
                    if (__any(hits != 0))   // most chunks hold no key
                        append(std::integral_constant<int, 1>(), &hits, &i, &c, &q[u], direct, cand);
                }
            }
        });
        ties = __builtin_amdgcn_readlane(wave_incl_scan(ties), 63);
        if (lane == 0) {
            if (i < d.n) {
                w.rowcnt[(int64_t)b * w.max_n + i] = ties;
                w.rowseg[(int64_t)b * w.max_n + i] = segs;
            }
            part[wv] = ties;
        }
        __syncthreads();
        if (tid == 0) w.blkcnt[(int64_t)b * w.nblk_stride + blk] = part[0] + part[1] + part[2] + part[3];
        __syncthreads();   // buf, nbuf, base and part are the next item's
    }
}

// ---------------------------------------------------------------- ordering

// Order the K pivots of one pair by (w desc, i asc, j asc) and write (i, j, w).
// Keys are distinct, so a key's rank is the number of smaller keys. Each
// workgroup of kSortWaves waves copies the pair's collected keys into its LDS
// and ranks 64 of them: wave v counts the smaller keys in its slice of the
// list with eight 16-byte broadcast reads in flight, and the partial counts
// are summed. The work of one pair is spread over ceil(K/64) CUs.
//
// Ordered path: the collected keys are the c_gt pairs heavier than alpha and
// fill slots 0 .. c_gt-1; slot c_gt + t holds the t-th pair of weight alpha in
// row-major order. A workgroup whose 64 slots reach past c_gt finds its ties
// from the row scan's counts: an exclusive scan of the per-block tie counts
// names the (at most 64) blocks that hold them, and one wave per block walks
// its rows' segments, counting ties in order, and writes those in its range.
constexpr int kSortWaves = 16;
constexpr int kSortThreads = 64 * kSortWaves;

__global__ void __launch_bounds__(kSortThreads) k_sort(Work w, int blocks_per_pair)
{
    extern __shared__ uint64_t keys[];
    __shared__ int32_t part[kSortWaves][64];
    __shared__ int64_t lds[17];
    __shared__ int32_t nrel, rel_blk[64], rel_pre[64];
    const int slot = blockIdx.x / blocks_per_pair, b = batch_pair(w, slot), g = blockIdx.x - slot * blocks_per_pair;
    const PairDesc d = pair_desc(w, b);
    const int K = d.kpiv, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // the collection counters are read together with the state (they are zeroed for every pair)
    int c[kCollectRegions];
#pragma unroll
    for (int r = 0; r < kCollectRegions; ++r) c[r] = w.tick[(int64_t)b * w.tick_stride + r * kTickLine];
    const PairState st = w.state[b];
    // the keys sit in the kCollectRegions regions of the pool, as many in each as its counter says
    int rb[kCollectRegions + 1];
    rb[0] = 0;
#pragma unroll
    for (int r = 0; r < kCollectRegions; ++r) rb[r + 1] = rb[r] + min(max(c[r], 0), w.pool_cap);
    // keys ranked (the first K are kept): fast path c_gt + all ties, ordered path c_gt
    const int want = K > 0 ? (st.fast ? st.ncand : st.c_gt) : 0;
    const int NC = min(min(want, rb[kCollectRegions]), w.pool_cap);
    int32_t *out = w.pivots_plain + (int64_t)b * w.pool_cap * 3;
    if (g * 64 >= max(NC, w.pool)) return;
    const uint64_t *cand = w.cand + (int64_t)b * kCollectRegions * w.pool_cap;
    const int K16 = (NC + 15) & ~15;   // padded with keys larger than any real one
    for (int k0 = tid; k0 < K16; k0 += kSortThreads * 8) {   // eight keys per thread loaded before any is stored
        uint64_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = k0 + kSortThreads * u;
            int r = 0, o = 0;   // the region holding key k and its first key (rb is non-decreasing)
#pragma unroll
            for (int q = 1; q < kCollectRegions; ++q)
                if (k >= rb[q]) { r = q; o = rb[q]; }
            v[u] = k < NC ? cand[(int64_t)r * w.pool_cap + (k - o)] : ~0ull;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (k0 + kSortThreads * u < K16) keys[k0 + kSortThreads * u] = v[u];
    }
    __syncthreads();
    const int p = g * 64 + lane;
    const uint64_t mine = p < NC ? keys[p] : 0;
    if (g * 64 < NC) {   // the same on the whole workgroup
        const int per = ((K16 / 16 + kSortWaves - 1) / kSortWaves) * 16;   // a slice of whole 16-key groups
        const int q0 = min(K16, wv * per), q1 = min(K16, q0 + per);
        int r = 0;
        for (int q = q0; q < q1; q += 16) {
            uint4 a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] = *reinterpret_cast<const uint4 *>(&keys[q + 2 * u]);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                r += (((uint64_t)a[u].y << 32) | a[u].x) < mine;
                r += (((uint64_t)a[u].w << 32) | a[u].z) < mine;
            }
        }
        part[wv][lane] = r;
        __syncthreads();
        if (wv == 0) {
            int rk = 0;
#pragma unroll
            for (int v = 0; v < kSortWaves; ++v) rk += part[v][lane];
            if (p < NC && rk < K) {
                out[3 * rk] = (int32_t)((mine >> 20) & 0xFFFFF);
                out[3 * rk + 1] = (int32_t)(mine & 0xFFFFF);
                out[3 * rk + 2] = (int32_t)(0xFFFFu - (uint32_t)(mine >> 40));
            }
        }
    }
    if (wv == 0 && p >= K && p < w.pool) {   // slots past the pair's pivots
        out[3 * p] = -1;
        out[3 * p + 1] = -1;
        out[3 * p + 2] = 0;
    }
    if (K <= 0 || st.fast) return;
    // ordered path: ties t0 .. t1-1 of this workgroup's slots
    const int cgt = st.c_gt, alpha = st.alpha;
    const int t0 = max(g * 64, cgt) - cgt, t1 = min(g * 64 + 64, K) - cgt;
    if (t1 <= t0) return;
    const int nblk = (d.n + kRowsPerItem - 1) / kRowsPerItem;
    const int32_t *bc = w.blkcnt + (int64_t)b * w.nblk_stride;
    int bcnt[8];
    int64_t local = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u) {   // blocks 8t .. 8t+7 per thread (nblk <= 8192)
        const int k = 8 * tid + u;
        bcnt[u] = k < nblk ? bc[k] : 0;
        local += bcnt[u];
    }
    if (tid == 0) nrel = 0;
    int64_t total;
    int64_t run = block_exclusive_scan<int64_t>(local, lds, total);   // its barriers order nrel's reset
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        if (bcnt[u] > 0 && run < t1 && run + bcnt[u] > t0) {   // the block holds a tie of the range
            const int slot = atomicAdd(&nrel, 1);
            if (slot < 64) {
                rel_blk[slot] = 8 * tid + u;
                rel_pre[slot] = (int32_t)run;
            }
        }
        run += bcnt[u];
    }
    __syncthreads();
    const int nr = min(nrel, 64);
    const uint16_t *G = w.G + d.g_off;
    const int c1 = (d.n + 7) >> 3;
    for (int x = wv; x < nr; x += kSortWaves) {
        int pre = rel_pre[x];
        const int blk = rel_blk[x];
        for (int rr = 0; rr < kRowsPerItem; ++rr) {
            const int i = blk * kRowsPerItem + rr;
            if (i >= d.n || pre >= t1) break;
            const int ne = w.rowcnt[(int64_t)b * w.max_n + i];
            if (ne > 0 && pre + ne > t0) {
                // the row's ties in order, eight segments (512 columns each) loaded at a time
                const uint16_t *row = G + (int64_t)i * d.npad;
                const int c_lo = (i + 1) >> 3;
                uint64_t todo = w.rowseg[(int64_t)b * w.max_n + i];
                int idx0 = pre;   // tie index of the row's next tie
                while (todo && idx0 < t1) {
                    uint4 q[8];
                    int cs[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        int cc = -1;
                        if (todo) {
                            cc = c_lo + 64 * __builtin_ctzll(todo) + lane;
                            todo &= todo - 1;
                        }
                        cs[u] = cc;
                        q[u] = (cc >= 0 && cc < c1) ? *reinterpret_cast<const uint4 *>(row + 8 * cc)
                                                    : make_uint4(0, 0, 0, 0);
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int cc = cs[u];
                        if (__builtin_amdgcn_readfirstlane(cc) < 0) break;   // no segment left (the same on every lane)
                        const int lo = min(max(i + 1 - 8 * cc, 0), 8), hi = min(max(d.n - 8 * cc, 0), 8);
                        const uint32_t uw[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
                        uint32_t heq = 0;
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            heq |= ((uint32_t)((int)(uw[k] & 0xFFFFu) == alpha) << (2 * k)) |
                                   ((uint32_t)((int)(uw[k] >> 16) == alpha) << (2 * k + 1));
                        heq &= ((1u << hi) - 1u) & ~((1u << lo) - 1u);
                        const int m = __builtin_popcount(heq);
                        const int incl = wave_incl_scan(m);
                        int idx = idx0 + incl - m;
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            if ((heq >> e) & 1u) {
                                if (idx >= t0 && idx < t1) {
                                    const int slot = cgt + idx;   // < K <= pool_cap
                                    out[3 * slot] = i;
                                    out[3 * slot + 1] = 8 * cc + e;
                                    out[3 * slot + 2] = alpha;
                                }
                                ++idx;
                            }
                        }
                        idx0 += __builtin_amdgcn_readlane(incl, 63);
                    }
                }
            }
            pre += ne;
        }
    }
}

}  // namespace

// grid_rows: workgroups of the row scan
hipError_t launch_pivots(const Work &w, int B, int grid_rows, int num_cus, hipStream_t s)
{
    if (w.n1 && w.n1 <= kFuseThreshMax) {
        hipLaunchKernelGGL(k_rowscan<true>, dim3(std::min(grid_rows, num_cus)), dim3(256), (size_t)w.n1 * sizeof(int32_t), s, w);
    } else {
        hipLaunchKernelGGL(k_thresh, dim3(B), dim3(1024), (size_t)w.max_n * sizeof(int32_t), s, w);
        hipLaunchKernelGGL(k_rowscan<false>, dim3(grid_rows), dim3(256), 0, s, w);
    }
    const int bpp = (w.pool_cap + 63) / 64;   // the fast path may rank up to pool_cap keys
    hipLaunchKernelGGL(k_sort, dim3(B * bpp), dim3(kSortThreads), (size_t)((w.pool_cap + 15) & ~15) * sizeof(uint64_t),
                       s, w, bpp);
    return hipGetLastError();
}

hipError_t setup_pivot_kernels()
{
    // up to TR_MAX_POOL keys (128 KiB) / 32767 histogram bins in LDS
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_sort),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, TR_MAX_POOL * (int)sizeof(uint64_t));
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_thresh), hipFuncAttributeMaxDynamicSharedMemorySize,
                                32768 * (int)sizeof(int32_t));
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_rowscan<true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kFuseThreshMax * (int)sizeof(int32_t));
    return e;
}

}  // namespace tr
