// Graph construction on gfx950: work planning, the pairwise-length
// compatibility matrix (Eq. 1) and the SC2 weights of the O2Graph
// (Eq. 2 restricted to i < j, Definition 2) on FP4 MFMA with exact float32 accumulation.
#include <algorithm>

#include "common.h"


namespace tr {
namespace {

__device__ __forceinline__ int wave_sum(int v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Upper-triangular tile index t (row-major over bi <= bj < nb) -> (bi, bj).
__device__ __forceinline__ void tri_decode(int t, int nb, int &bi, int &bj)
{
    // start(r) = r*(2nb - r + 1)/2 tiles precede row r
    float a = (float)(2 * nb + 1);
    int r = (int)((a - sqrtf(a * a - 8.0f * (float)t)) * 0.5f);
    r = r < 0 ? 0 : (r >= nb ? nb - 1 : r);
    while (r > 0 && r * (2 * nb - r + 1) / 2 > t) --r;
    while (r + 1 < nb && (r + 1) * (2 * nb - r) / 2 <= t) ++r;
    bi = r;
    bj = r + (t - r * (2 * nb - r + 1) / 2);
}

// SC2 tile order: the upper triangle of nb x nb tiles is walked in super-tiles
// of sup x sup (super-rows I <= J, row-major), tiles row-major inside.
// Consecutive items then share few row blocks of C, so the tiles one XCD runs
// at the same time reuse each other's operand rows in its L2. sup >= 1 is a
// launch parameter (the autotuner's); the order does not change any result.
__device__ __forceinline__ void super_decode(int t, int nb, int sup, int &bi, int &bj)
{
    // a super-row holds whole tile rows, so the tiles before it are those before its first row
    tri_decode(t, nb, bi, bj);
    const int I = bi / sup, r0 = I * sup, s = min(nb, r0 + sup) - r0;
    t -= r0 * (2 * nb - r0 + 1) / 2;
    if (t < s * (s + 1) / 2) {   // the diagonal super-tile, a triangle of side s
        tri_decode(t, s, bi, bj);
        bi += r0;
        bj += r0;
        return;
    }
    t -= s * (s + 1) / 2;
    const int J = t / (s * sup), c0 = r0 + sup * (J + 1), c = min(nb, c0 + sup) - c0;   // only the last is narrower
    t -= J * s * sup;
    bi = r0 + t / c;
    bj = c0 + t % c;
}

// ---------------------------------------------------------------- planning

// Exclusive scan of NV values per thread across the workgroup (one pass).
template <int NV>
__device__ void block_scan_multi(const int64_t (&v)[NV], int64_t (&excl)[NV], int64_t (&total)[NV],
                                 int64_t (*lds)[NV])
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    int64_t x[NV];
#pragma unroll
    for (int s = 0; s < NV; ++s) {
        x[s] = v[s];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t y = __shfl_up(x[s], o, 64);
            if (lane >= o) x[s] += y;
        }
        if (lane == 63) lds[wid][s] = x[s];
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        int64_t acc = 0;
        for (int k = 0; k < nw; ++k) { const int64_t t = lds[k][threadIdx.x]; lds[k][threadIdx.x] = acc; acc += t; }
        lds[nw][threadIdx.x] = acc;
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < NV; ++s) {
        excl[s] = lds[wid][s] + x[s] - v[s];
        total[s] = lds[nw][s];
    }
    __syncthreads();
}

constexpr int kCostKeys = 32767 / kSc2Tile + 2;   // npad / kSc2Tile of a valid pair (max_n <= 32767), 0 if invalid
constexpr int kOrderMinB = 16;   // smaller batches keep their pairs in index order

// Slot of the pair at position p of the size order (largest first) among B pairs: the order is
// dealt to the eight XCDs in a snake (positions 0-7 to XCDs 0-7, 8-15 to XCDs 7-0, ...), and the
// slots hold XCD 0's pairs, then XCD 1's, ..., each XCD's pairs in size order. Cut into eight
// ranges of equal cost, the SC2 list then gives each XCD a like mix of sizes, costly items first.
__device__ __forceinline__ int xcd_pairs(int x, int B)
{
    const int R = B >> 3, rem = B & 7;
    return R + (rem && ((R & 1) ? x >= 8 - rem : x < rem));
}

__device__ __forceinline__ int xcd_first_slot(int x, int B)
{
    int first = 0;
    for (int y = 0; y < x; ++y) first += xcd_pairs(y, B);
    return first;
}

__device__ __forceinline__ int snake_slot(int p, int B)
{
    const int r = p >> 3, c = p & 7;
    return xcd_first_slot((r & 1) ? 7 - c : c, B) + r;
}

// One workgroup: per-pair sizes, arena offsets (pair order) and zeroed per-pair state; the
// order of the pairs (from 16 pairs on: by decreasing npad, pairs of one size in index order,
// dealt to the XCDs; else index order);
// the work-item counts of every stage and their prefix sums over that order; the XCD ranges of
// the SC2 list, equal in modelled cost; the launch shapes that follow the pairs' own sizes
// (the sizes a batch is declared for may be far above them).
__global__ void __launch_bounds__(1024) k_plan(const int32_t *offsets, int32_t n_single, int32_t B,
                                               int32_t max_n, int32_t pool, int32_t H, int32_t num_cus, bool sparse,
                                               PairDesc *pairs, PairState *state, Plan *plan,
                                               int32_t *pre, int32_t pre_stride, uint8_t *masks)
{
    constexpr int NV = kNumPrefix + 1;   // the work-list stages, then the SC2 cost
    __shared__ int64_t lds[17][NV];
    __shared__ int64_t lds1[17][2];
    __shared__ int32_t kfirst[kCostKeys];        // pairs per size key, then the key's next free position
    __shared__ int32_t wfirst[16][kCostKeys];    // per wave of a chunk: pairs per key, then first position
    __shared__ int32_t nl[1024], ol[1024];       // B <= 1024: n of each valid pair (0 if invalid); the order
    __shared__ int32_t sp_tiles[kSpEdges];       // bit-count tiles of each edge over all pairs (sparse_tile)
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, nw = blockDim.x >> 6;
    int32_t *order = pre + kOrderRow * pre_stride, *slot_of = pre + kSlotRow * pre_stride;
    auto size_of = [&](int b, int32_t &n, int32_t &pt) {   // n and first match of pair b; valid?
        n = pt = 0;
        if (b >= B) return false;
        if (offsets) { pt = offsets[b]; n = offsets[b + 1] - pt; }
        else n = n_single;
        return n >= 3 && n <= max_n;
    };
    const bool small = B <= 1024;
    auto valid_n = [&](int b) {   // n of pair b if it is valid, else 0 (passes 2 and 3)
        if (b >= B) return 0;
        if (small) return nl[b];
        int32_t n, pt;
        return size_of(b, n, pt) ? n : 0;
    };
    // modelled cost of one SC2 item in K columns of its main loop: npad columns, plus the
    // epilogue (scan, histogram, stores), which takes about as long as 2048 columns
    auto sc2_unit = [](int32_t npad) { return (int64_t)npad + 2048; };
    for (int k = tid; k < kCostKeys; k += blockDim.x) kfirst[k] = 0;
    if (tid < kSpEdges) sp_tiles[tid] = 0;
    __syncthreads();
    // pass 1, pair order: descriptors, state, arena offsets, size-key counts, total SC2 cost
    int64_t acarry = 0, sc2_cost = 0;
    for (int base = 0; base < B; base += blockDim.x) {
        const int b = base + tid;
        int32_t n, pt;
        const bool ok = size_of(b, n, pt);
        const int32_t npad = ok ? (n + kSc2Tile - 1) / kSc2Tile * kSc2Tile : 0;
        int64_t v[2] = {(int64_t)npad * npad, ok ? stage_items(kSc2, n, H, 0) * sc2_unit(npad) : 0}, excl[2], tot[2];
        block_scan_multi<2>(v, excl, tot, lds1);
        if (b < B) {
            PairDesc d = pair_desc_of(n, pt, excl[0] + acarry, pool);
            if (!ok) d.n = d.npad = d.kpiv = 0;
            pairs[b] = d;
            PairState st = {};
            st.status = ok ? TR_OK : TR_ERR_INVALID_ARG;
            if (masks && n < 3)   // no other kernel writes the mask of such a pair
                for (int k = 0; k < n; ++k) masks[pt + k] = 0;
            state[b] = st;
            atomicAdd(&kfirst[npad / kSc2Tile], 1);
            if (small) nl[b] = ok ? n : 0;
            if (ok && sparse)
                for (int k = 0; k < kSpEdges; ++k) atomicAdd(&sp_tiles[k], (int)stage_items(kSp, n, H, 256 * (k + 1)));
        }
        acarry += tot[0];
        sc2_cost += tot[1];
    }
    __syncthreads();
    if (B < kOrderMinB) {   // a few pairs: slots in pair order
        for (int b = tid; b < B; b += blockDim.x) {
            order[b] = slot_of[b] = b;
            if (small) ol[b] = b;
        }
    } else {
        {   // first position of each key, the largest key first
            int64_t v[2] = {tid < kCostKeys ? kfirst[kCostKeys - 1 - tid] : 0, 0}, excl[2], tot[2];
            block_scan_multi<2>(v, excl, tot, lds1);
            if (tid < kCostKeys) kfirst[kCostKeys - 1 - tid] = (int32_t)excl[0];
            __syncthreads();
        }
        // pass 2, pair order: positions (pairs of one key in index order: rank in the wave by
        // ballots, then the waves of the chunk in order), and slots
        for (int base = 0; base < B; base += blockDim.x) {
            const int b = base + tid;
            const int key = (valid_n(b) + kSc2Tile - 1) / kSc2Tile;
            const int nwa = min(nw, (B - base + 63) >> 6);   // waves of the chunk that hold pairs
            for (int k = tid; k < nwa * kCostKeys; k += blockDim.x) (&wfirst[0][0])[k] = 0;
            __syncthreads();
            bool pending = b < B;
            int rank = 0;
            uint64_t todo = __ballot(pending);
            while (todo) {
                const int lk = __builtin_amdgcn_readlane(key, __builtin_ctzll(todo));
                const bool mine = pending && key == lk;
                const uint64_t m = __ballot(mine);
                if (mine) {
                    rank = __builtin_popcountll(m & ((1ull << lane) - 1));
                    pending = false;
                }
                if (lane == 0) wfirst[wid][lk] = __builtin_popcountll(m);
                todo &= ~m;
            }
            __syncthreads();
            for (int k = tid; k < kCostKeys; k += blockDim.x) {
                int32_t acc = kfirst[k];
                for (int v = 0; v < nwa; ++v) {
                    const int32_t c = wfirst[v][k];
                    wfirst[v][k] = acc;
                    acc += c;
                }
                kfirst[k] = acc;
            }
            __syncthreads();
            if (b < B) {
                const int slot = snake_slot(wfirst[wid][key] + rank, B);
                order[slot] = b;
                slot_of[b] = slot;
                if (small) ol[slot] = b;
            }
            __syncthreads();   // wfirst is cleared next chunk
        }
    }
    __syncthreads();   // order[] is read by other threads below
    // pass 3, slot order: stage prefixes; SC2 range boundaries at x / 8 of the cost
    const int32_t sp = sparse ? sparse_tile(sp_tiles, num_cus) : 0;
    if (tid == 0) {
        plan->B = B;
        plan->sp_tile = sp;
        plan->sc2_split[0] = 0;
        for (int x = 1; x < 8; ++x)
            if (sc2_cost * x / 8 == 0) plan->sc2_split[x] = 0;
    }
    int64_t carry[NV] = {};
    for (int base = 0; base < B; base += blockDim.x) {
        const int slot = base + tid;
        const int b = slot >= B ? B : small ? ol[slot] : order[slot];
        const int32_t n = valid_n(b);
        const bool ok = n > 0;
        int64_t cnt[NV], excl[NV], tot[NV];
        for (int s = 0; s < kNumPrefix; ++s) cnt[s] = ok ? stage_items(s, n, H, sp) : 0;
        cnt[kScore] = ok ? cnt[kScore] : (b < B);   // an invalid pair's one (empty) scoring item writes its record
        const int32_t npad = ok ? (n + kSc2Tile - 1) / kSc2Tile * kSc2Tile : 0;
        cnt[kNumPrefix] = ok ? cnt[kSc2] * sc2_unit(npad) : 0;
        block_scan_multi<NV>(cnt, excl, tot, lds);
        if (slot < B) {
            for (int s = 0; s < kNumPrefix; ++s) pre[s * pre_stride + slot] = (int32_t)(excl[s] + carry[s]);
            // a target in (c0, c1] falls in this pair's items: the first item whose cost prefix reaches it
            const int64_t c0 = excl[kNumPrefix] + carry[kNumPrefix], c1 = c0 + cnt[kNumPrefix];
            for (int x = 1; x < 8; ++x) {
                const int64_t tgt = sc2_cost * x / 8;
                if (tgt > c0 && tgt <= c1) {
                    const int64_t u = sc2_unit(npad);
                    plan->sc2_split[x] = (int32_t)(excl[kSc2] + carry[kSc2] + (tgt - c0 + u - 1) / u);
                }
            }
        }
#pragma unroll
        for (int s = 0; s < NV; ++s) carry[s] += tot[s];
    }
    if (tid == 0) {
        for (int s = 0; s < kNumPrefix; ++s) {
            pre[s * pre_stride + B] = (int32_t)carry[s];
            plan->total[s] = (int32_t)carry[s];
        }
        plan->sc2_split[8] = (int32_t)carry[kSc2];
        plan->compat_rows = compat_rows(carry[kCompat], num_cus);
    }
}

// ---------------------------------------------------------------- Eq. 1

typedef float v16f __attribute__((ext_vector_type(16)));


// A value that is the same on every lane, in scalar registers.
__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Exchange of the wave's halves: a' = [a of lanes 0-31, b of lanes 0-31], b' = [a of 32-63, b of 32-63].
__device__ __forceinline__ void swap_halves(uint32_t &a, uint32_t &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

// Maximum over the wave of values >= 0 (as integers they order alike), in every lane.
__device__ __forceinline__ float wave_fmax(float v)
{
    int m = __float_as_int(v);
    m = max(m, __builtin_amdgcn_update_dpp(0, m, 0x111, 0xf, 0xf, false));   // row_shr:1
    m = max(m, __builtin_amdgcn_update_dpp(0, m, 0x112, 0xf, 0xf, false));   // row_shr:2
    m = max(m, __builtin_amdgcn_update_dpp(0, m, 0x114, 0xf, 0xf, false));   // row_shr:4
    m = max(m, __builtin_amdgcn_update_dpp(0, m, 0x118, 0xf, 0xf, false));   // row_shr:8
    m = max(m, __builtin_amdgcn_update_dpp(0, m, 0x142, 0xa, 0xf, false));   // row_bcast:15 into rows 1, 3
    m = max(m, __builtin_amdgcn_update_dpp(0, m, 0x143, 0xc, 0xf, false));   // row_bcast:31 into rows 2, 3
    return __int_as_float(__builtin_amdgcn_readlane(m, 63));
}

// One step of a 32 x 32 bit transpose across the 32 lanes of each half of the wave: lanes S apart
// exchange the bits whose position differs in S (M: the positions with that bit clear).
template <int S, uint32_t M>
__device__ __forceinline__ uint32_t transpose_step(uint32_t x, int lane)
{
    const uint32_t y = (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, (S << 10) | 0x1f);   // lane ^ S
    const bool hi = lane & S;
    const uint32_t z = __builtin_amdgcn_alignbit(y, y, hi ? S : 32 - S), mk = hi ? M : ~M;
    return (z & mk) | (x & ~mk);
}

// Bit r of lane c becomes bit c of lane r, in each half of the wave.
__device__ __forceinline__ uint32_t transpose32(uint32_t x, int lane)
{
    x = transpose_step<16, 0x0000FFFFu>(x, lane);
    x = transpose_step<8, 0x00FF00FFu>(x, lane);
    x = transpose_step<4, 0x0F0F0F0Fu>(x, lane);
    x = transpose_step<2, 0x33333333u>(x, lane);
    return transpose_step<1, 0x55555555u>(x, lane);
}

// C of 8 to 128 rows x 128 columns per work item, one wave per item and no workgroup barrier: a lane
// holds two columns' points in registers, the rows' points (R <= 32 at a time) are broadcast from LDS (the
// next row's read ahead), and each pair is evaluated once for both triangles. Off the diagonal an item
// writes its rows and their transpose. A lane's decisions collect as one bit per row, so a column is an
// R-bit word (the transpose's R / 8 bytes) and a bit transpose across lanes gives the rows' 16 bytes.
//
// With a = |x_i - x_j|^2, b = |y_i - y_j|^2, s = a + b, d = a - b, L = sqrt a + sqrt b, the test
// |sqrt a - sqrt b| <= tau is for s >= tau^2 the sign of E = d^2 - 2 tau^2 s + tau^4 =
// (delta^2 - tau^2)(L^2 - tau^2): no square root, and the sign bit shifts straight into the lane's word
// (20 issue slots a pair; 26 with two hardware square roots). A guard makes every decision the exact one
// (length32, correctly rounded roots). Both sides take the same float a and b; the exact evaluation's roots and
// difference move delta by at most e = 2^-23 L, so E at its decision is at most e (2 tau + e)(L^2 - tau^2) off zero:
// 2^-21 tau L s, and 2^-44 s^2 where rounding alone exceeds tau (scenes 10^8 times larger and more). E's own
// rounding is 2^-22 of these terms and of tau^2 s. The boundary report counts |delta - tau| < 1e-6: with e + 1e-6
// for e, 4e-6 tau s and 4e-12 s more in E (the second where tau is below 1e-6 or so).
// A row holding a pair with |E| <= tau s (2^-18 L + 5e-6) + 5e-12 s + 2^-42 s^2 + 2.1 tau^4 is evaluated exactly
// (L^2 <= 2 s, L <= s / L0 + L0 / 2 for any L0; the last term covers the pairs with s near or below tau^2, where E's
// sign says nothing). Items with a non-finite or huge point (beyond 1e8), and thresholds outside [1e-9, 1e8], are
// evaluated exactly throughout.
//
// Counts (edges, boundary pairs, non-finite input; the last by diagonal items) go to the item's slot. The
// diagonal items clear the pair's weight histograms for their rows, and with learned pivots
// the row marks.
__global__ void __launch_bounds__(256) k_compat(Work w)
{
    __shared__ float4 rows[4][32][2];
    __shared__ SlotCache slots;
    if (w.sp_list && blockIdx.x == 0 && threadIdx.x < 2) w.sp_list[threadIdx.x] = 0;   // counted up by k_sc2_sparse
    const bool cached = slot_cache_fill(w, kCompat, slots);
    __syncthreads();
    const int ROWS = __builtin_amdgcn_readfirstlane(compat_item_rows(w)), R = min(ROWS, 32), per = kCompatTile / ROWS, total = stage_total(w, kCompat) * per;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float tau = w.tau, t2 = 2.0f * tau * tau, t4 = (tau * tau) * (tau * tau);
    const bool odd_tau = !(tau >= 1e-9f && tau <= 1e8f);
    if (w.n1 && blockIdx.x == 0)   // its counters (collection regions, clique-search tickets)
        for (int k = tid; k < w.tick_stride / kTickLine; k += 256) w.tick[k * kTickLine] = 0;
    if (w.n1 && blockIdx.x == 0 && tid == 0) {   // a single-pair call has no planner: reset its state here
        PairState st = {};
        st.status = TR_OK;
        w.state[0] = st;
    }
    for (int item = blockIdx.x * 4 + wv; item < total; item += gridDim.x * 4) {
        int local, bi, bj;
        const int tile = item / per;
        const int b = __builtin_amdgcn_readfirstlane(stage_pair_cached(w, kCompat, slots, cached, tile, local));
        const PairDesc d = pair_desc(w, b);
        const int n = __builtin_amdgcn_readfirstlane(d.n), npad = __builtin_amdgcn_readfirstlane(d.npad);
        local = __builtin_amdgcn_readfirstlane(local);
        tri_decode(local, npad / kCompatTile, bi, bj);
        bi = __builtin_amdgcn_readfirstlane(bi);
        bj = __builtin_amdgcn_readfirstlane(bj);
        const int j0 = bj * kCompatTile + lane;
        const bool diag = bi == bj;
        const float *src = w.src + 3 * (int64_t)d.pt_off, *dst = w.dst + 3 * (int64_t)d.pt_off;
        // past n a copy of the last point, whose decisions are masked
        float3 x[2], y[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int jc = min(j0 + 64 * c, n - 1);
            x[c] = *reinterpret_cast<const float3 *>(src + 3 * jc);
            y[c] = *reinterpret_cast<const float3 *>(dst + 3 * jc);
        }
        auto wild_point = [](float3 q) { return !(__builtin_fabsf(q.x) + __builtin_fabsf(q.y) + __builtin_fabsf(q.z) < 1e8f); };
        const bool wild_col = odd_tau || __any(wild_point(x[0]) || wild_point(x[1]) || wild_point(y[0]) || wild_point(y[1]));
        float near_at[2];   // a lane past n is never near
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            near_at[c] = j0 + 64 * c < n ? 2.1f * t4 : -1.0f;
            asm volatile("" : "+v"(near_at[c]));   // kept in its register, not formed again for each row
        }
        uint8_t *Cb = w.C + uniform64(d.c_off) / 8;
        const uint32_t kbs = (uint32_t)npad * 16;   // bytes of one 128-column block over all rows
        int nbnd = 0, nedge = 0;
        bool any_bad = false;
        const int first = (item - tile * per) * ROWS;   // the item's first row in the tile
#pragma unroll 1
        for (int rof = first; rof < first + ROWS; rof += R) {
            const int i0 = bi * kCompatTile + rof;
            // lanes 0-31 stage the rows' source points, lanes 32-63 their targets
            const int ri = i0 + (lane & 31);
            const float3 p = *reinterpret_cast<const float3 *>((lane >> 5 ? dst : src) + 3 * min(ri, n - 1));
            const bool bad = diag && (lane & 31) < R && ri < n && !(isfinite(p.x) && isfinite(p.y) && isfinite(p.z));
            rows[wv][lane & 31][lane >> 5] = make_float4(p.x, p.y, p.z, 0.0f);
            const bool wild = wild_col || __any(wild_point(p));
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int nr = min(R, n - i0);   // rows below n
            const int top = max((nr + 1) & ~1, 0) - 1;   // rows in pairs from the last one; one past n is masked
            float4 a1 = rows[wv][max(top, 0)][0], q1 = rows[wv][max(top, 0)][1];
            // L0: the largest |x_i - x_j| of one row, so that L0 is near the L of most pairs
            const float lx = a1.x - x[0].x, ly = a1.y - x[0].y, lz = a1.z - x[0].z;
            const float L0 = fmaxf(2.0f * __builtin_amdgcn_sqrtf(wave_fmax(wild ? 0.0f : lx * lx + ly * ly + lz * lz)), 16.0f * tau);
            const float g1 = __builtin_fmaf(tau, 0x1p-18f / L0, 0x1p-42f);
            const float g0 = __builtin_fmaf(tau, __builtin_fmaf(L0, 0x1p-19f, 5e-6f), 5e-12f);
            uint64_t self[2] = {0, 0};   // diagonal tile: the lane holding row 0's own match
            if (diag) self[rof >> 6] = 1ull << (rof & 63);
            uint32_t col[2] = {0, 0};    // bit r: pair (i0 + r, j)
            auto row = [&](int r, const float4 &a, const float4 &q) {
                float E[2];
                uint64_t near = 0;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const float ax = a.x - x[c].x, ay = a.y - x[c].y, az = a.z - x[c].z;
                    const float bx = q.x - y[c].x, by = q.y - y[c].y, bz = q.z - y[c].z;
                    float s1 = ax * ax, s2 = bx * bx;
                    s1 = __builtin_fmaf(ay, ay, s1);
                    s2 = __builtin_fmaf(by, by, s2);
                    s1 = __builtin_fmaf(az, az, s1);
                    s2 = __builtin_fmaf(bz, bz, s2);
                    const float df = s1 - s2, s = s1 + s2;
                    E[c] = __builtin_fmaf(df, df, -__builtin_fmaf(t2, s, -t4));
                    near |= __ballot(__builtin_fmaf(-__builtin_fmaf(g1, s, g0), s, __builtin_fabsf(E[c])) <= near_at[c]) &
                            ~(self[c] << r);
                }
                if (wild || near) {
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const float l1 = length32(a.x - x[c].x, a.y - x[c].y, a.z - x[c].z);
                        const float l2 = length32(q.x - y[c].x, q.y - y[c].y, q.z - y[c].z);
                        const float dl = __builtin_fabsf(l1 - l2);
                        E[c] = dl <= tau ? -1.0f : 1.0f;
                        const int j = j0 + 64 * c;
                        if (i0 + r < j && j < n && r < nr) nbnd += __builtin_fabsf(dl - tau) < 1e-6f;
                    }
                }
#pragma unroll
                for (int c = 0; c < 2; ++c) col[c] = __builtin_amdgcn_alignbit(col[c], __float_as_uint(E[c]), 31);
            };
            for (int r = top; r > 0; r -= 2) {
                const float4 a0 = rows[wv][r - 1][0], q0 = rows[wv][r - 1][1];
                row(r, a1, q1);
                a1 = rows[wv][max(r - 2, 0)][0];
                q1 = rows[wv][max(r - 2, 0)][1];
                row(r - 1, a0, q0);
            }
            const uint32_t live = nr >= 32 ? 0xFFFFFFFFu : nr <= 0 ? 0u : (1u << nr) - 1u;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int j = j0 + 64 * c, k = j - i0;   // diagonal tile: rows r < k lie above it, r == k on it
                col[c] = j < n ? col[c] & live : 0u;
                if (diag && k >= 0 && k < 32) col[c] &= ~(1u << k);
                nedge += __builtin_popcount(!diag ? col[c] : k <= 0 ? 0u : k >= 32 ? col[c] : col[c] & ((1u << k) - 1u));
            }
            if (!diag) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    uint8_t *o = Cb + (uint32_t)bi * kbs + (uint32_t)(j0 + 64 * c) * 16 + rof / 8;
                    if (R == 32) *reinterpret_cast<uint32_t *>(o) = col[c];
                    else if (R == 16) *reinterpret_cast<uint16_t *>(o) = (uint16_t)col[c];
                    else *o = (uint8_t)col[c];
                }
            }
            // lane (r, h): columns 32 h .. of row r in c0, 64 + 32 h .. in c1; the halves' exchange leaves words
            // 2 h and 2 h + 1 of the row's four
            uint32_t c0 = transpose32(col[0], lane), c1 = transpose32(col[1], lane);
            swap_halves(c0, c1);
            if ((lane & 31) < R)
                *reinterpret_cast<uint2 *>(Cb + (uint32_t)bj * kbs + (uint32_t)(i0 + (lane & 31)) * 16 + 8 * (lane >> 5)) =
                    make_uint2(c0, c1);
            any_bad = any_bad || __any(bad);
            if (diag && (lane & 31) < R && ri < n) {
#pragma unroll
                for (int g = 0; g < kHistGroups; g += 2)
                    w.ghist[((int64_t)b * kHistGroups + g + (lane >> 5)) * w.hist_stride + ri] = 0;
                const int64_t rw = (int64_t)b * w.max_n + ri;
                if (w.learned && lane < 32) w.mark[rw] = 0;   // the row marks
            }
        }
        const int sums = wave_sum((nbnd << 15) | nedge);   // at most 16384 pairs each
        if (lane == 0) w.cnt_part[item] = (uint32_t)sums | ((uint32_t)any_bad << 30);
    }
}

// The same matrix with the features' accumulators (training): per match the degree and a 16-bin
// histogram of delta over all other matches. A lane holds one row's point and the columns' points are
// broadcast from LDS, so each row's counts stay with its lane (an LDS word per bin and lane, which its own
// lane alone updates in a wave: no conflicts and no atomics in memory) and its bits of C shift into words
// in place. Every pair is evaluated from both sides (twice the arithmetic of the triangle), which cost less
// than adding the columns' counts across lanes: 598 us for 64 pairs of 1000 to 5000 matches; 64 x 64 tiles
// with LDS histograms of rows and columns, added in memory, and correctly rounded roots throughout took 1549.
//
// Bins: t = delta / q (q = tau / 4) with the hardware square roots; a pair whose delta lies within
// 2^-19 (|x| + |y|) + 2e-6 + 2^-17 q of the nearest bin edge (tau is edge 4; |y| <= |x| + 4 tau there) is
// evaluated again with the correctly rounded ones, so every bin and bit is the exact one. One workgroup per
// 64 rows (a quarter of a list item of kPrepRows rows), the 64-column blocks dealt to its waves; the sums
// are written whole.
constexpr int kFeatWaves = 8;
__global__ void __launch_bounds__(64 * kFeatWaves) k_compat_features(Work w)
{
    __shared__ float4 cols[kFeatWaves][64][2];
    __shared__ int32_t hist[16][64], deg[64];
    if (w.sp_list && blockIdx.x == 0 && threadIdx.x < 2) w.sp_list[threadIdx.x] = 0;   // counted up by k_sc2_sparse
    const int total = (kPrepRows / 64) * stage_total(w, kPrep);
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float tau = w.tau, q = tau * 0.25f, inv_q = 1.0f / q;
    const float band0 = __builtin_fmaf(tau, 0x1p-17f, __builtin_fmaf(q, 0x1p-17f, 2.1e-6f));
    for (int item = blockIdx.x; item < total; item += gridDim.x) {
        int local;
        const int b = __builtin_amdgcn_readfirstlane(stage_pair(w, kPrep, item / (kPrepRows / 64), local));
        const PairDesc d = pair_desc(w, b);
        const int n = __builtin_amdgcn_readfirstlane(d.n), npad = __builtin_amdgcn_readfirstlane(d.npad);
        const int i0 = __builtin_amdgcn_readfirstlane(local) * kPrepRows + 64 * (item % (kPrepRows / 64)), i = i0 + lane;
        const float *src = w.src + 3 * (int64_t)d.pt_off, *dst = w.dst + 3 * (int64_t)d.pt_off;
        const float3 x = *reinterpret_cast<const float3 *>(src + 3 * min(i, n - 1));
        const float3 y = *reinterpret_cast<const float3 *>(dst + 3 * min(i, n - 1));
        for (int k = tid; k < 16 * 64; k += 64 * kFeatWaves) hist[k >> 6][k & 63] = 0;
        if (tid < 64) deg[tid] = 0;
        __syncthreads();
        __attribute__((address_space(3))) int32_t *h = (__attribute__((address_space(3))) int32_t *)&hist[0][lane];
        uint8_t *Cb = w.C + uniform64(d.c_off) / 8 + (uint32_t)i * 16;
        const uint32_t kbs = (uint32_t)npad * 16;   // bytes of one 128-column block over all rows
        int degree = 0;
        const int nblk = npad / 64;
        float3 px, py;   // the next block's points: lane's column
        auto fetch = [&](int blk) {
            const int jc = min(64 * blk + lane, n - 1);
            px = *reinterpret_cast<const float3 *>(src + 3 * jc);
            py = *reinterpret_cast<const float3 *>(dst + 3 * jc);
        };
        fetch(min(wv, nblk - 1));
        for (int blk = wv; blk < nblk; blk += kFeatWaves) {
            const int j0 = 64 * blk, cnt = i0 < n ? min(64, n - j0) : 0;   // columns below n
            __builtin_amdgcn_wave_barrier();   // the block before is read
            cols[wv][lane][0] = make_float4(px.x, px.y, px.z, 0.0f);
            cols[wv][lane][1] = make_float4(py.x, py.y, py.z, 0.0f);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (blk + kFeatWaves < nblk) fetch(blk + kFeatWaves);
            uint32_t word[2] = {0, 0};
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                uint32_t W = 0;
                const int top = min(32, cnt - 32 * g) - 1;
                float4 na = cols[wv][max(32 * g + top, 0)][0], nq = cols[wv][max(32 * g + top, 0)][1];
#pragma unroll 2
                for (int c = top; c >= 0; --c) {
                    const float4 a = na, r = nq;
                    na = cols[wv][32 * g + max(c - 1, 0)][0];
                    nq = cols[wv][32 * g + max(c - 1, 0)][1];
                    const float ax = a.x - x.x, ay = a.y - x.y, az = a.z - x.z;
                    const float bx = r.x - y.x, by = r.y - y.y, bz = r.z - y.z;
                    float s1 = ax * ax, s2 = bx * bx;
                    s1 = __builtin_fmaf(ay, ay, s1);
                    s2 = __builtin_fmaf(by, by, s2);
                    s1 = __builtin_fmaf(az, az, s1);
                    s2 = __builtin_fmaf(bz, bz, s2);
                    const float la = __builtin_amdgcn_sqrtf(s1), lb = __builtin_amdgcn_sqrtf(s2);
                    float dl = __builtin_fabsf(la - lb);
                    const float t = dl * inv_q;
                    const float kn = __builtin_amdgcn_fmed3f(__builtin_rintf(t), 1.0f, 15.0f);
                    int bin = (int)__builtin_fminf(t, 15.0f);
                    // not clearly outside the band: also a NaN (a non-finite point; bin 0, no edge)
                    const bool near = !(__builtin_fabsf(__builtin_fmaf(-kn, q, dl)) > __builtin_fmaf(la, 0x1p-18f, band0));
                    if (__any(near)) {
                        if (near) {
                            dl = __builtin_fabsf(length32(ax, ay, az) - length32(bx, by, bz));
                            bin = 0;
#pragma unroll
                            for (int k = 1; k < 16; ++k) bin += dl >= (float)k * q;
                        }
                    }
                    W = (W << 1) | (dl <= tau ? 1u : 0u);
                    __hip_atomic_fetch_add(h + 64 * bin, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                const int k = i - j0 - 32 * g;   // a match with itself has no entry
                if (k >= 0 && k < 32) W &= ~(1u << k);
                word[g] = i < n ? W : 0u;
                degree += __builtin_popcount(word[g]);
            }
            *reinterpret_cast<uint2 *>(Cb + (uint32_t)(blk >> 1) * kbs + 8 * (blk & 1)) = make_uint2(word[0], word[1]);
        }
        atomicAdd(&deg[lane], degree);
        // the match itself was counted as any other: out of its bin again (delta 0: the last where the bins have no width;
        // the first also if it is not finite)
        const float self = (x.x - x.x) + (x.y - x.y) + (x.z - x.z) + (y.x - y.x) + (y.y - y.y) + (y.z - y.z);   // 0 or NaN
        if (wv == 0) atomicAdd(&hist[self >= q ? 15 : 0][lane], -1);
        __syncthreads();
        // slots: 0 degree, 3 .. 18 the histogram, the others padding (the SC2 sum and maximum come as parts)
        int32_t *rs = w.rowstat + ((int64_t)b * w.max_n + i0) * 20;
        for (int k = tid; k < 64 * 20 && i0 + k / 20 < n; k += 64 * kFeatWaves) {
            const int r = k / 20, f = k % 20;
            rs[k] = f == 0 ? deg[r] : f < 3 || f == 19 ? 0 : hist[f - 3][r];
        }
        __syncthreads();   // hist and deg are the next item's
    }
}

// ---------------------------------------------------------------- Eq. 2 on FP4 MFMA

typedef int32_t v8i __attribute__((ext_vector_type(8)));
typedef int32_t v16i __attribute__((ext_vector_type(16)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) void gvoid;
typedef __attribute__((address_space(3))) void lvoid;

constexpr int kOut = 128;                      // output tile edge: four waves of 64 x 64
// Weights 1 .. kHistLdsBins are histogrammed in LDS first (weight v in word v - 1). Behind the bins: a
// spare word per lane of a wave, and the tile's largest weight (two slots used in turn).
constexpr int kHistLdsBins = 8126;
constexpr int kHistWords = kHistLdsBins + 64 + 2;
constexpr int kHistBytes = kHistWords * 4;
constexpr int kOutPitch = kOut + 8;            // uint16 per LDS row of a tile staged for the column statistics
constexpr int kOutBytes = kOut / 2 * kOutPitch * 2;   // half of its rows at a time
constexpr float kAccBias = 8388608.0f;         // 2^23: a count v < 2^16 is then the low 16 bits of 2^23 + v
// What the epilogue leaves besides the weights: the histogram and segment maxima the pivots need, the
// row sums and maxima the learned features need, or both (a learned registration).
enum Sc2Mode { kSc2Plain = 0, kSc2Learned = 1, kSc2Features = 2 };
constexpr int kSc2PerCu = 3;                   // workgroups resident per CU (registers: 168 per lane; two took 64 feature
                                               // pairs from 615 to 650 us, learned N = 5000 from 34.9 to 38.5)

// Maximum over each half of the wave (lanes 0-31, 32-63), left in lanes 31 and 63: prefix
// steps inside each 16-lane DPP row, then the last lane of rows 0 and 2 joins rows 1 and 3.
// Inputs are >= 0, so lanes that receive no value (they read 0) do not change a maximum.
__device__ __forceinline__ int half_max(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false));   // row_shr:1
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false));   // row_shr:2
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false));   // row_shr:4
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false));   // row_shr:8
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));   // row_bcast:15 into rows 1, 3
    return v;
}

// Add the workgroup's LDS histogram of weights 1 .. top into the pair's global copy and clear it.
// Called by all threads after a barrier.
__device__ __forceinline__ void hist_flush(int32_t *hist, int32_t *gh, int top)
{
    for (int k = threadIdx.x; k < top; k += blockDim.x) {
        const int c = hist[k];
        if (c) {
            atomicAdd(&gh[k + 1], c);
            hist[k] = 0;
        }
    }
}

// hist[k] += 1 as an LDS instruction (through a generic pointer the compiler may emit a flat atomic).
__device__ __forceinline__ void lds_add(int32_t *hist, uint32_t k)
{
    __hip_atomic_fetch_add((__attribute__((address_space(3))) int32_t *)hist + k, 1, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Sums and maxima of the tile's columns (column j of the upper tile is row j of the lower one, the
// SC2 matrix being symmetric), from half of the masked tile's rows at a time in LDS: thread t takes columns 2c,
// 2c+1 (c = t mod 64) over rows of one residue class (its wave), sixteen 4-byte reads in flight; the classes
// meet in xl (3 ints per column pair and class), which may overlie the rows.
struct ColumnStats {
    int s0 = 0, s1 = 0;
    u16x2 mx = {0, 0};

    __device__ __forceinline__ void add(const uint16_t *T)   // after a barrier
    {
        const uint32_t *Tw = reinterpret_cast<const uint32_t *>(T) + (threadIdx.x >> 6) * (kOutPitch / 2) + (threadIdx.x & 63);
        uint32_t v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = Tw[4 * u * (kOutPitch / 2)];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            s0 += (int)(v[u] & 0xFFFFu);
            s1 += (int)(v[u] >> 16);
            mx = __builtin_elementwise_max(mx, __builtin_bit_cast(u16x2, v[u]));
        }
    }

    // csum, cmax: the tile's first column there, its groups of 32 columns `stride` apart
    __device__ __forceinline__ void store(int32_t *xl, int32_t *csum, uint16_t *cmax, int stride)   // after a barrier
    {
        const int cp = threadIdx.x & 63, cls = threadIdx.x >> 6;
        if (cls) {
            int32_t *x = xl + 3 * ((cls - 1) * 64 + cp);
            x[0] = s0;
            x[1] = s1;
            x[2] = (int32_t)__builtin_bit_cast(uint32_t, mx);
        }
        __syncthreads();
        if (!cls) {
#pragma unroll
            for (int c = 1; c < 4; ++c) {
                const int32_t *x = xl + 3 * ((c - 1) * 64 + cp);
                s0 += x[0];
                s1 += x[1];
                mx = __builtin_elementwise_max(mx, __builtin_bit_cast(u16x2, (uint32_t)x[2]));
            }
            const int at = cp / 16 * stride + 2 * cp % 32;
            *reinterpret_cast<int2 *>(csum + at) = make_int2(s0, s1);
            *reinterpret_cast<uint32_t *>(cmax + at) = __builtin_bit_cast(uint32_t, mx);
        }
    }
};

// One 128 x 128 output tile (bi <= bj in units of 128) of G[i][j] = C_ij sum_k C_ik C_jk, i < j < n,
// by a workgroup of four waves in a 2 x 2 layout, each a 64 x 64 sub-tile of 2 x 2 blocks of
// v_mfma_scale_f32_32x32x64_f8f6f4 with FP4 (E2M1) operands. C is symmetric, so the product is C C^T
// and both operands are rows of C read along k.
//
// C is stored as bits and becomes FP4 in registers. A lane's 16-byte piece of a row (128 k) holds
// bit p of every nibble p = 0..3; the four operands (w & 0x1111.., w & 0x2222.., w & 0x4444..,
// (w >> 3) & 0x1111..) are then E2M1 0.5, 1, 2 and 0.5 where the bit is set, and the E8M0 block
// scales (x 2, 1, 1/2, 2 on each side) make every product 0 or 1. Which k a nibble stands for does
// not matter as both operands take the same order. Every partial sum is an integer below 2^24, so
// the float32 accumulation is exact. Accumulators start at 2^23: a finished count is the low 16 bits
// of the float. Operands come straight from L2 in whole 512-byte runs (lanes 0-31 the 32 rows' piece
// of one 128-column block, lanes 32-63 of the next), two steps of 256 k in flight, with no LDS and no
// barrier in the loop: a quarter of the bytes of nibbles in memory, and the epilogue of one
// workgroup runs under the products of the CU's other ones. At N = 5000 the kernel takes 33.6 us
// (58.3 with 256 x 256 tiles fed as nibbles through an LDS ring, one workgroup per CU), at N = 1000
// 7.0 (29.6), at N = 20000 1220 (1890): 6.6 PFLOP/s of the 7.8 that FP4 products alone sustain here.
// Four workgroups per CU (128 registers) changed nothing; the rest at N = 5000 is the last, partly
// filled round of tiles (820 tiles over 256 CUs) and 4.5 us of stores of the weights.
//
// The operands are swapped (A: rows j, B: rows i), so a lane's 16 accumulators of a block are one row
// i; two swaps between the wave's halves make them two runs of eight consecutive columns. Each run
// is masked by the row's bits of C, stored with one 16-byte write (whole runs: outside i < j < n they
// hold zeros, which nothing reads), counted into the LDS weight histogram and reduced into the row
// maximum.
template <int MODE>
__device__ __forceinline__ void sc2_dense_tile(const Work &w, const PairDesc &d, int b, int bi, int bj, int copy,
                                               int32_t *hist, int32_t *tmax, uint16_t *T)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, wm = wv >> 1, wn = wv & 1;
    const int l31 = lane & 31, lh = lane >> 5;
    const uint8_t *Cb = w.C + uniform64(d.c_off) / 8;
    const uint32_t kbs = (uint32_t)__builtin_amdgcn_readfirstlane(d.npad) * 16;   // bytes of one 128-column block over all rows
    const int ns = (int)(kbs >> 12);              // steps of 256 k
    const int i0 = bi * kOut + wm * 64, j0 = bj * kOut + wn * 64;
    const uint32_t oj = lh * kbs + (uint32_t)(j0 + l31) * 16, oi = lh * kbs + (uint32_t)(i0 + l31) * 16;
    // the rows' bits of C over the wave's 64 columns (block bj), used after the products
    const auto rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(Cb), 0, kbs * (uint32_t)(2 * ns), 0x00027000);
    uint2 cm[2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
        cm[x] = *reinterpret_cast<const uint2 *>(Cb + (uint32_t)bj * kbs + (uint32_t)(i0 + 32 * x + l31) * 16 + wn * 8);
    v16f acc[2][2];   // [i block][j block]
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[x][y][r] = kAccBias;
    // (buffer loads: the step is a scalar offset)
    auto load = [&](int s, v4u (&fj)[2], v4u (&fi)[2]) {
        const int so = sc2_step_offset(s, ns, kbs);
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            fj[y] = __builtin_amdgcn_raw_buffer_load_b128(rows, oj + y * 512, so, 0);
            fi[y] = __builtin_amdgcn_raw_buffer_load_b128(rows, oi + y * 512, so, 0);
        }
    };
    auto step = [&](const v4u (&fj)[2], const v4u (&fi)[2]) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint32_t m = t == 1 ? 0x22222222u : t == 2 ? 0x44444444u : 0x11111111u;
            const int sh = t == 3 ? 3 : 0, scale = t == 1 ? 127 : t == 2 ? 126 : 128;
            v8i a[2], c[2];
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                a[y] = v8i{(int)((fj[y].x >> sh) & m), (int)((fj[y].y >> sh) & m), (int)((fj[y].z >> sh) & m),
                           (int)((fj[y].w >> sh) & m), 0, 0, 0, 0};
                c[y] = v8i{(int)((fi[y].x >> sh) & m), (int)((fi[y].y >> sh) & m), (int)((fi[y].z >> sh) & m),
                           (int)((fi[y].w >> sh) & m), 0, 0, 0, 0};
            }
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y)
                    acc[x][y] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[y], c[x], acc[x][y], 4, 4, 0, scale,
                                                                                 0, scale);
        }
    };
    v4u j_a[2], i_a[2], j_b[2], i_b[2];
    load(0, j_a, i_a);
    load(1, j_b, i_b);
    int s = 0;
    for (; s + 1 < ns; s += 2) {
        step(j_a, i_a);
        load(s + 2, j_a, i_a);
        __builtin_amdgcn_sched_barrier(0);   // keep the two steps' loads apart: one is always in flight
        step(j_b, i_b);
        load(s + 3, j_b, i_b);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (s < ns) step(j_a, i_a);
    // ---- epilogue: lane (l31, lh) of block (x, y) holds row i0 + 32x + l31 and, after the swaps, columns
    // j0 + 32y + 16q + 8 lh .. + 7 for q = 0, 1
    int32_t *gh = w.ghist + ((int64_t)b * kHistGroups + copy) * w.hist_stride;
    uint16_t *Gb = w.G + d.g_off;
    const bool small_n = d.n <= kHistLdsBins + 1;
    const uint32_t spare = kHistLdsBins + lane;
    int wmax = 0;
    ColumnStats cols;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const int i = i0 + 32 * x + l31;
        u16x2 rm = {0, 0};
        int rs = 0;
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            uint32_t cw = y ? cm[x].y : cm[x].x;   // C_ij of columns j0 + 32y + e at bit e
            if (bi == bj) {                        // i < j only
                const int k = i - (j0 + 32 * y);
                cw &= k < 0 ? 0xFFFFFFFFu : k >= 31 ? 0u : 0xFFFFFFFEu << k;
            }
            cw >>= 8 * lh;
            const v16i ai = __builtin_bit_cast(v16i, acc[x][y]);
            uint32_t p[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) p[k] = __builtin_amdgcn_perm(ai[2 * k + 1], ai[2 * k], 0x05040100);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                uint32_t o[4] = {p[4 * q], p[4 * q + 1], p[4 * q + 2], p[4 * q + 3]};
                swap_halves(o[0], o[2]);
                swap_halves(o[1], o[3]);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t lo = (uint32_t)((int32_t)(cw << (31 - 16 * q - 2 * k)) >> 31);
                    const uint32_t hi = (uint32_t)((int32_t)(cw << (30 - 16 * q - 2 * k)) >> 31);
                    o[k] &= (lo & 0xFFFFu) | (hi & 0xFFFF0000u);
                    rm = __builtin_elementwise_max(rm, __builtin_bit_cast(u16x2, o[k]));
                    if (MODE != kSc2Plain) rs += (int)((o[k] & 0xFFFFu) + (o[k] >> 16));
                }
                const int jc = j0 + 32 * y + 16 * q + 8 * lh;
                *reinterpret_cast<uint4 *>(Gb + (int64_t)i * d.npad + jc) = make_uint4(o[0], o[1], o[2], o[3]);
                if (MODE != kSc2Plain)
                    *reinterpret_cast<uint4 *>(&T[(32 * wm + l31) * kOutPitch + jc - bj * kOut]) =
                        make_uint4(o[0], o[1], o[2], o[3]);
                if (MODE != kSc2Features) {
                    // no branch: a zero entry (v - 1 wraps) and one past the LDS bins count in the lane's
                    // own spare word, so zeros do not queue at one address
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        lds_add(hist, min((o[k] & 0xFFFFu) - 1u, spare));
                        lds_add(hist, min((o[k] >> 16) - 1u, spare));
                    }
                    if (!small_n) {   // the same on the whole workgroup
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            if ((o[k] & 0xFFFFu) > kHistLdsBins) atomicAdd(&gh[o[k] & 0xFFFFu], 1);
                            if ((o[k] >> 16) > kHistLdsBins) atomicAdd(&gh[o[k] >> 16], 1);
                        }
                    }
                }
            }
        }
        uint32_t m0 = (uint32_t)max((int)rm.x, (int)rm.y), m1 = m0;
        swap_halves(m0, m1);
        const int m = max((int)m0, (int)m1);
        wmax = max(wmax, m);
        if (MODE != kSc2Plain) {
            uint32_t r0 = (uint32_t)rs, r1 = r0;
            swap_halves(r0, r1);
            rs = (int)(r0 + r1);
        }
        if (lh == 0) {
            // parts that the readers add up: atomics on the rows' totals (and the columns' below) took 16 of 53 us at
            // N = 5000 and 150 of 800 us for 64 feature pairs
            const int64_t at = d.g_off / 64 + part_at(i, j0 / 64, d.npad / 64);
            w.segmax[at] = (uint16_t)m;
            if (MODE != kSc2Plain) w.rowsum[at] = rs;
        }
        if (MODE != kSc2Plain) {
            __syncthreads();   // this half of the rows is in T
            cols.add(T);
            __syncthreads();   // T is the other half's, or the classes'
        }
    }
    if (MODE != kSc2Features) {
        wmax = half_max(wmax);   // both halves of the wave hold the same rows
        if (lane == 31) atomicMax(tmax, wmax);
    }
    __syncthreads();   // T, the histogram and the tile's maximum are complete
    if (MODE != kSc2Features) {
        const int top = *tmax;   // the pair's largest weight stands in bin 0 of the copies
        if (threadIdx.x == 0 && top > 0) atomicMax(&gh[0], top);
        hist_flush(hist, gh, min(top, kHistLdsBins));
    }
    if (MODE != kSc2Plain) {
        const int64_t at = d.g_off / 128 + part_at(bj * kOut, bi, d.npad / kOut);
        cols.store(reinterpret_cast<int32_t *>(T), w.colsum + at, w.colmax + at, d.npad / kOut * 32);
    }
}

// This workgroup's share of the SC2 list in 256 x 256 tiles: XCD x takes a contiguous range of the
// list (neighbouring tiles share rows of C in its L2): equal counts for one pair, equal shares of the
// modelled cost for a batch.
__device__ __forceinline__ void sc2_range(const Work &w, int &start, int &end)
{
    const int xcd = blockIdx.x & 7;
    if (w.n1) {
        const int total = stage_total(w, kSc2), chunk = (total + 7) >> 3;
        start = xcd * chunk;
        end = min(total, start + chunk);
    } else {
        start = w.plan->sc2_split[xcd];
        end = w.plan->sc2_split[xcd + 1];
    }
}

// Dense product of every tile: a work item is one 128 x 128 quadrant of a list tile (quadrants below
// the diagonal or past n are skipped).
template <int MODE>
__global__ void __launch_bounds__(256, kSc2PerCu) k_sc2(Work w)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    int32_t *hist = reinterpret_cast<int32_t *>(smem), *tmax = hist + kHistWords - 2;   // zero outside the epilogue
    uint16_t *T = reinterpret_cast<uint16_t *>(smem + (MODE == kSc2Features ? 0 : kHistBytes));
    int start, end;
    const int nx = (gridDim.x - (blockIdx.x & 7) + 7) >> 3, sp = w.sp_list ? sc2_sparse_edge(w) : 0, m = sp / kOut;
    if (sp) {   // the tiles that the bit-count kernel left, dealt to the XCDs
        start = 0;
        end = (w.sp_list[0] - (int)(blockIdx.x & 7) + 7) / 8 * m * m;
    } else {
        sc2_range(w, start, end);
        start *= 4;
        end *= 4;
    }
    if (MODE != kSc2Features)
        for (int k = threadIdx.x; k < kHistWords / 4; k += 256) reinterpret_cast<int4 *>(hist)[k] = make_int4(0, 0, 0, 0);
    __syncthreads();
    int par = 0;
    for (int it = start + (blockIdx.x >> 3); it < end; it += nx) {
        int local, b, bi, bj;
        if (sp) {
            const int q = it % (m * m);
            b = stage_pair(w, kSp, w.sp_list[2 + it / (m * m) * 8 + (blockIdx.x & 7)], local);
            tri_decode(local, (pair_desc(w, b).n + sp - 1) / sp, bi, bj);
            bi = __builtin_amdgcn_readfirstlane(m * bi + q / m);
            bj = __builtin_amdgcn_readfirstlane(m * bj + q % m);
        } else {
            b = stage_pair(w, kSc2, it >> 2, local);
            super_decode(local, pair_desc(w, b).npad / kSc2Tile, w.sc2_super, bi, bj);
            bi = __builtin_amdgcn_readfirstlane(2 * bi + ((it >> 1) & 1));
            bj = __builtin_amdgcn_readfirstlane(2 * bj + (it & 1));
        }
        const PairDesc d = pair_desc(w, b);
        if (bi > bj || bj * kOut >= d.n) continue;   // the same for the whole workgroup
        sc2_dense_tile<MODE>(w, d, b, bi, bj, it % kHistGroups, hist, &tmax[par], T);
        if (MODE != kSc2Features && threadIdx.x == 0) tmax[par ^ 1] = 0;   // read before this tile's barrier, written after the next
        par ^= 1;
        __syncthreads();   // the histogram is clear, T is the next item's
    }
}

// ---- the same weights by counting bits, for tiles with few edges
//
// Eq. 2 is needed only where C_ij = 1, so an S x S tile (S = 256 .. 1024) with few edges counts
// popcount(row_i AND row_j) for each of them. The rows' bits stream through LDS in 128-column blocks, S rows of
// I and S rows of J, 16 bytes each, one block counted and three in flight. Edges are listed row by row in runs
// of four of one row; a thread holds up to five runs, packed LDS offsets and counts in registers, and per block
// and run reads row i's piece once and four rows j. More runs than the threads hold take another pass over the
// rows. Of sixteen waves one feeds the buffers (its waits count its own loads, so stores never stand before a
// block), one writes the tile's zeros to G meanwhile, fourteen count; then the weights are stored over the zeros
// and go to the histogram and the row statistics, which take the buffers' place in LDS. Tiles with too many
// edges go to a list that k_sc2 works off next.
//
// What bounds it: the LDS reads of rows j, 16 lanes at a time at random rows of 16 bank groups, on average three
// deep (counters: 10.6 cycles an instruction, 4 without conflicts; N = 20000 has 250 of its 330 us per tile in
// them). Measured at 1.3 % edges: N = 20000 375 us where k_sc2 takes 1230, sixteen such pairs 4.6 ms (18.7 ms with
// 256 x 256 tiles, edges in 64-byte pieces and a tile staged in LDS for the store). Software-pipelined reads with
// a barrier per two blocks: 395; all sixteen waves feeding, zeroing and counting: 392; a read of row i per edge
// where it changes instead of runs: 618 (16 edges a thread). Ordering a row's edges by bank class would meet 3 to
// 10 % fewer conflicts, an order that knows the other lanes' 24 %, for about the time it saves.
constexpr int kSpThreads = 1024, kSpWaves = kSpThreads / 64;
constexpr int kSpCount = 14 * 64;                  // threads of the counting waves
constexpr int kRuns = 5;                           // runs per counting thread: four edges of one row each
constexpr int kSpCap = kSpCount * kRuns;           // runs of a pass
constexpr int kSpMax = 1024;                       // largest tile edge
constexpr int kSpSide = kSpMax * 16;               // one block's rows of I or J
constexpr int kSpBufs = 4;                         // blocks in LDS: one counted, three in flight
constexpr int kSpRing = kSpBufs * 2 * kSpSide;     // before and after the counting other data
constexpr int kSpStat = kHistBytes;                // learned statistics: column maxima, row and column sums
// Weights up to kSpLow (most, where a tile has few edges) count in copies by lane: on few bins 64 lanes' adds queue.
constexpr int kSpLow = 255, kSpCopies = 16, kSpPitch = kSpLow + 2;
constexpr int kSpLowAt = kSpStat + 3 * kSpMax * 4;
constexpr int kSpSegAt = kSpLowAt + kSpCopies * kSpPitch * 4;    // maxima by 64-column segment and row
constexpr int kSpZero = kSpSegAt / 4 + kSpMax / 64 * kSpMax;     // words cleared before the weights are collected
constexpr int kSpLds = kSpRing + 8 * kSpWaves + 16;
static_assert(kSpCap * 16 <= kSpRing && 4 * kSpZero <= kSpRing && kSpZero % 4 == 0, "LDS layout of the bit-count kernel");
static_assert(kSpMax == 256 * kSpEdges, "tile edges of the bit-count kernel");

// Wait until at most n vector-memory operations of this wave are outstanding (n is rounded down).
__device__ __forceinline__ void wait_vm(int n)
{
    if (n >= 56) asm volatile("s_waitcnt vmcnt(56)" ::: "memory");
    else if (n >= 48) asm volatile("s_waitcnt vmcnt(48)" ::: "memory");
    else if (n >= 32) asm volatile("s_waitcnt vmcnt(32)" ::: "memory");
    else if (n >= 16) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
    else if (n >= 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// BATCH: the tile edge is the plan's; a single pair's is a kernel argument (read from memory, N = 20000 took 611 us a
// call, 604 so).
template <int MODE, bool BATCH>
__global__ void __launch_bounds__(kSpThreads) k_sc2_sparse(Work w)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    typedef __attribute__((address_space(3))) const uint8_t lds8;
    typedef __attribute__((address_space(3))) const v4u ldsv;
    int32_t *hist = reinterpret_cast<int32_t *>(smem), *tmax = hist + kHistWords - 2;
    int32_t *cmax = reinterpret_cast<int32_t *>(smem + kSpStat), *rsum = cmax + kSpMax, *csum = rsum + kSpMax;
    int32_t *seg = reinterpret_cast<int32_t *>(smem + kSpSegAt);
    int32_t *scan = reinterpret_cast<int32_t *>(smem + kSpRing);
    uint32_t *list = reinterpret_cast<uint32_t *>(smem);
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int total = stage_total(w, kSp);
    for (int item = blockIdx.x, next; item < total; item = next) {
        const int S = BATCH ? __builtin_amdgcn_readfirstlane(w.plan->sp_tile) : w.sp_tile;
        int local;
        const int b = __builtin_amdgcn_readfirstlane(stage_pair(w, kSp, item, local));
        const PairDesc d = pair_desc(w, b);
        const int n = __builtin_amdgcn_readfirstlane(d.n), npad = __builtin_amdgcn_readfirstlane(d.npad);
        local = __builtin_amdgcn_readfirstlane(local);
        int bi, bj;
        tri_decode(local, (n + S - 1) / S, bi, bj);
        bi = __builtin_amdgcn_readfirstlane(bi);
        bj = __builtin_amdgcn_readfirstlane(bj);
        const bool diag = bi == bj;
        const int i0 = bi * S, j0 = bj * S, nkb = npad / 128;
        const uint8_t *Cb = w.C + uniform64(d.c_off) / 8;
        const uint32_t kbs = (uint32_t)npad * 16;   // bytes of one 128-column block over all rows
        // ---- the tile's edges: thread t has row i0 + t over the tile's columns
        int row = tid;
        asm volatile("" : "+v"(row));   // what depends on it is not kept over the tiles: registers are short
        const bool has_row = row < S && i0 + row < npad;
        auto row_bits = [&](int kb) {   // the row's 128 columns j0 + 128 kb ..; on the diagonal tile i < j only
            v4u v = {0, 0, 0, 0};
            if (has_row && 128 * kb < S && j0 + 128 * kb < npad) {
                v = *reinterpret_cast<const v4u *>(Cb + (uint32_t)(j0 / 128 + kb) * kbs + (uint32_t)(i0 + row) * 16);
                if (diag) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int k = row - 128 * kb - 32 * e;   // bits above the row's own
                        v[e] &= k < 0 ? 0xFFFFFFFFu : k >= 31 ? 0u : 0xFFFFFFFEu << k;
                    }
                }
            }
            return v;
        };
        int mine = 0;
#pragma unroll
        for (int kb = 0; kb < kSpMax / 128; ++kb) {
            const v4u v = row_bits(kb);
            mine += __builtin_popcount(v.x) + __builtin_popcount(v.y) + __builtin_popcount(v.z) + __builtin_popcount(v.w);
        }
        const int runs = (mine + 3) / 4;
        int incl = runs, sum = mine;   // inclusive scan of the runs inside the wave, then the waves before
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
            sum += __shfl_xor(sum, o, 64);
        }
        if (lane == 63) {
            scan[2 * wv] = incl;
            scan[2 * wv + 1] = sum;
        }
        if (tid == 0) scan[2 * kSpWaves] = gridDim.x + atomicAdd(&w.sp_list[1], 1);   // whoever is free takes the next tile
        __syncthreads();
        int first = incl - runs, all = 0, edges = 0;
#pragma unroll
        for (int v = 0; v < kSpWaves; ++v) {
            const int c = scan[2 * v];
            first += v < wv ? c : 0;
            all += c;
            edges += scan[2 * v + 1];
        }
        next = __builtin_amdgcn_readfirstlane(scan[2 * kSpWaves]);
        all = __builtin_amdgcn_readfirstlane(all);
        edges = __builtin_amdgcn_readfirstlane(edges);
        // (counted against the whole square, the half tiles on the diagonal and the narrow last ones of pairs too dense
        // for this kernel came here, up to two passes of 20 CUs alone: 1738 us a call at N = 20000, 5.3 %; 1389 now)
        const int entries = min(S, n - i0) * min(S, n - j0) / (diag ? 2 : 1);   // the last tiles are narrower
        const bool take = edges <= (entries + 255) / 256 * w.sp_cap / 256;   // sp_cap of every 65536
        if (!take) {   // the same for the whole workgroup: the dense kernel's
            if (tid == 0) w.sp_list[2 + atomicAdd(&w.sp_list[0], 1)] = item;
            __syncthreads();
            continue;
        }
        uint16_t *Gb = w.G + d.g_off;
        int32_t *gh = w.ghist + ((int64_t)b * kHistGroups + local % kHistGroups) * w.hist_stride;
        // zeros of the tile: rows from, from + step, .. below to (a wave), up to column npad
        const int zrows = min(S, n - i0), zcols = min(S, npad - j0);
        auto zeros = [&](int from, int to, int step) {
            for (int r = from; r < to; r += step) {
                uint16_t *p = Gb + (int64_t)(i0 + r) * npad + j0;
                for (int c = 8 * lane; c < zcols; c += 512) *reinterpret_cast<uint4 *>(p + c) = make_uint4(0, 0, 0, 0);
            }
        };
        // learned statistics of row i0 + t and column j0 + t (rs, cs: sums, cm: maximum; `more`: beyond those stored
        // already): the tile's sums stand in one of its segments that the row has, zeros in the others
        auto tile_stats = [&](int rs, int cs, int cm, bool more) {
            const int own = diag ? tid / 64 : 0;
            for (int v = 0; v < S / 64; ++v)
                if (i0 + tid < npad && j0 + 64 * v < npad) {
                    int32_t *p = w.rowsum + d.g_off / 64 + part_at(i0 + tid, j0 / 64 + v, npad / 64);
                    if (v == own) *p = more ? *p + rs : rs;
                    else if (!more) *p = 0;
                }
            for (int v = 0; v < S / 128; ++v)
                if (j0 + tid < npad && i0 + 128 * v < npad) {
                    const int64_t at = d.g_off / 128 + part_at(j0 + tid, i0 / 128 + v, npad / 128);
                    if (v == 0) {
                        w.colsum[at] = more ? w.colsum[at] + cs : cs;
                        w.colmax[at] = (uint16_t)(more ? max(cm, (int)w.colmax[at]) : cm);
                    } else if (!more) {
                        w.colsum[at] = 0;
                        w.colmax[at] = 0;
                    }
                }
        };
        for (int base = 0; base < all; base += kSpCap) {
            const int np = min(kSpCap, all - base);   // runs of this pass
            {
                int pos = 4 * (first - base);
                const int end = pos + 4 * runs;
                if (pos < 4 * np && end > 0) {
                    uint32_t e = 0;   // 16 row << 16 | 16 column, bit 31: an edge, not the filling of a run
                    v4u next = row_bits(0);
#pragma unroll 1
                    for (int kb = 0; kb < S / 128; ++kb) {
                        const v4u v = next;
                        next = row_bits(kb + 1);
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            uint32_t x = v[c];
                            while (x) {
                                e = (uint32_t)row << 20 | (uint32_t)(128 * kb + 32 * c + __builtin_ctz(x)) << 4 | 0x80000000u;
                                x &= x - 1;
                                if (pos >= 0 && pos < 4 * np) list[pos] = e;
                                ++pos;
                            }
                        }
                    }
                    for (; pos < end; ++pos)
                        if (pos >= 0 && pos < 4 * np) list[pos] = e & 0x7FFFFFFFu;
                }
            }
            __syncthreads();
            // counting thread t holds runs t q .. t q + q - 1 of the pass
            const int q = (np + kSpCount - 1) / kSpCount, r0 = min(np, tid * q), nr = tid < kSpCount ? min(q, np - r0) : 0;
            uint32_t ed[4 * kRuns], cnt[4 * kRuns];
#pragma unroll
            for (int k = 0; k < kRuns; ++k) {
                const v4u v = k < nr ? *reinterpret_cast<const v4u *>(list + 4 * (r0 + k)) : v4u{0, 0, 0, 0};
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    ed[4 * k + u] = v[u];
                    cnt[4 * k + u] = 0;
                }
            }
            __syncthreads();   // the list's room is the buffers'
            // at block kb's barrier the block has landed (wave 14 waited) and the reads of block kb - 1 are done
            if (wv == kSpWaves - 2) {
                // 64-row pieces of I and of J below npad (a multiple of 256), 1 KiB a load
                const int ends[2] = {min(S, npad - i0) * 16, min(S, npad - j0) * 16}, loads = (ends[0] + ends[1]) / 1024;
                auto feed = [&](int kb) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint8_t *p = Cb + (uint32_t)kb * kbs + (uint32_t)(h ? j0 : i0) * 16;
                        uint8_t *buf = smem + (kb % kSpBufs) * (2 * kSpSide) + h * kSpSide;
#pragma unroll 4
                        for (int v = 0; v < ends[h]; v += 1024)
                            __builtin_amdgcn_global_load_lds((gvoid *)(p + v + (uint32_t)lane * 16), (lvoid *)(buf + v), 16, 0, 0);
                    }
                };
                feed(0);
                feed(1);   // npad is a multiple of 256: at least two blocks
                if (nkb > 2) feed(2);
                for (int kb = 0; kb < nkb; ++kb) {
                    wait_vm(min(2, nkb - 1 - kb) * loads);
                    asm volatile("s_barrier" ::: "memory");
                    if (kb + 3 < nkb) feed(kb + 3);
                }
            } else if (wv == kSpWaves - 1) {
                const int zstep = (zrows + nkb - 1) / nkb;
                for (int kb = 0; kb < nkb; ++kb) {
                    asm volatile("s_barrier" ::: "memory");
                    if (base == 0) zeros(kb * zstep, min(zrows, (kb + 1) * zstep), 1);
                }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // in L2 before any weight is stored over them
            } else {
                for (int kb = 0; kb < nkb; ++kb) {
                    lds8 *buf = (lds8 *)smem + (kb % kSpBufs) * (2 * kSpSide);
                    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
                    for (int k = 0; k < kRuns; ++k) {
                        if (k < q) {   // uniform
                            const v4u ri = *(ldsv *)(buf + ((ed[4 * k] >> 16) & 0x7FFFu));
                            v4u rj[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u) rj[u] = *(ldsv *)(buf + (ed[4 * k + u] & 0xFFFFu) + kSpSide);
#pragma unroll
                            for (int u = 0; u < 4; ++u)
#pragma unroll
                                for (int e = 0; e < 4; ++e)
                                    asm("v_bcnt_u32_b32 %0, %1, %0" : "+v"(cnt[4 * k + u]) : "v"(ri[e] & rj[u][e]));
                        }
                    }
                }
            }
            __syncthreads();
            for (int k = tid; k < kSpZero / 4; k += kSpThreads) reinterpret_cast<int4 *>(smem)[k] = make_int4(0, 0, 0, 0);
            __syncthreads();
            int32_t *low = reinterpret_cast<int32_t *>(smem + kSpLowAt);
            const uint32_t copy = (uint32_t)(lane & (kSpCopies - 1)) * kSpPitch;
#pragma unroll
            for (int k = 0; k < kRuns; ++k) {
                const int i = (int)(ed[4 * k] >> 20) & (kSpMax - 1);
                int rs = 0;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t c = (int32_t)ed[4 * k + u] < 0 ? cnt[4 * k + u] : 0u;
                    const int j = (int)(ed[4 * k + u] >> 4) & (kSpMax - 1);
                    if (c > 0) {
                        Gb[(int64_t)(i0 + i) * npad + j0 + j] = (uint16_t)c;
                        atomicMax(&seg[(j >> 6) * kSpMax + i], (int)c);
                        if (MODE != kSc2Features) {   // the weight histogram counts nonzero weights
                            if (c <= (uint32_t)kSpLow) lds_add(low, copy + c);
                            else if (c <= (uint32_t)kHistLdsBins) lds_add(hist, c - 1);
                            else atomicAdd(&gh[c], 1);
                        }
                        if (MODE != kSc2Plain) {
                            atomicAdd(&csum[j], (int)c);
                            atomicMax(&cmax[j], (int)c);
                        }
                    }
                    rs += (int)c;
                }
                if (MODE != kSc2Plain && rs > 0) atomicAdd(&rsum[i], rs);
            }
            __syncthreads();
            // ---- the pass's row statistics and histogram
            if (MODE != kSc2Features && tid > 0 && tid <= kSpLow) {
                int c = 0;
#pragma unroll
                for (int v = 0; v < kSpCopies; ++v) c += low[v * kSpPitch + tid];
                hist[tid - 1] = c;   // no other add reached these bins
            }
            if (tid < S) {
                int m = 0;
                for (int v = 0; v < S / 64; ++v) {
                    const int x = seg[v * kSpMax + tid];
                    m = max(m, x);
                    if (i0 + tid < npad && j0 + 64 * v < npad) {
                        uint16_t *sm = w.segmax + d.g_off / 64 + part_at(i0 + tid, j0 / 64 + v, npad / 64);
                        *sm = (uint16_t)(base == 0 ? x : max(x, (int)*sm));
                    }
                }
                if (MODE != kSc2Features && m > 0) atomicMax(tmax, m);
                if (MODE != kSc2Plain) tile_stats(rsum[tid], csum[tid], cmax[tid], base > 0);
            }
            __syncthreads();
            if (MODE != kSc2Features) {
                const int top = *tmax;
                if (tid == 0 && top > 0) atomicMax(&gh[0], top);
                hist_flush(hist, gh, min(top, kHistLdsBins));
            }
            __syncthreads();   // the LDS is the next pass's
        }
        if (all == 0) {
            zeros(wv, zrows, kSpWaves);
            for (int v = 0; v < S / 64; ++v)
                if (tid < S && i0 + tid < npad && j0 + 64 * v < npad)
                    w.segmax[d.g_off / 64 + part_at(i0 + tid, j0 / 64 + v, npad / 64)] = 0;
            if (MODE != kSc2Plain && tid < S) tile_stats(0, 0, 0, false);
            __syncthreads();   // scan is the next tile's
        }
    }
}

}  // namespace

hipError_t launch_plan(const Work &w, const int32_t *offsets, int32_t n_single, int32_t B, int32_t max_n, int num_cus,
                       PairDesc *pairs, PairState *state, Plan *plan, int32_t *pre, hipStream_t s)
{
    hipLaunchKernelGGL(k_plan, dim3(1), dim3(1024), 0, s, offsets, n_single, B, max_n, w.pool, w.H,
                       num_cus, w.sp_list != nullptr, pairs, state, plan, pre, w.pre_stride, w.masks);
    return hipGetLastError();
}

// tiles: 128 x 128 tiles of the list; cap: workgroups to launch at most.
hipError_t launch_compat(const Work &w, int64_t tiles, int cap, hipStream_t s)
{
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((tiles * (kCompatTile / w.compat_rows) + 3) / 4, cap));
    hipLaunchKernelGGL(k_compat, dim3(grid), dim3(256), 0, s, w);
    return hipGetLastError();
}

// items: kPrepRows-row items of the list; cap: workgroups to launch at most.
hipError_t launch_compat_features(const Work &w, int64_t items, int cap, hipStream_t s)
{
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(items * (kPrepRows / 64), cap));
    hipLaunchKernelGGL(k_compat_features, dim3(grid), dim3(64 * kFeatWaves), 0, s, w);
    return hipGetLastError();
}

namespace {
constexpr int sc2_lds(int mode)
{
    return (mode == kSc2Features ? 0 : kHistBytes) + (mode == kSc2Plain ? 0 : kOutBytes);
}
}  // namespace

// Tiles of the bit-count kernel, before launch_sc2 takes those it left. tiles: of its list, at most.
hipError_t launch_sc2_sparse(const Work &w, int64_t tiles, int num_cus, hipStream_t s)
{
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(tiles, num_cus));
    const auto kernel = w.feat_all && w.learned ? k_sc2_sparse<kSc2Features, true>   // (features come in batches)
                        : w.learned ? w.n1 ? k_sc2_sparse<kSc2Learned, false> : k_sc2_sparse<kSc2Learned, true>
                        : w.n1 ? k_sc2_sparse<kSc2Plain, false> : k_sc2_sparse<kSc2Plain, true>;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kSpThreads), kSpLds, s, w);
    return hipGetLastError();
}

// items: 256 x 256 tiles of the list. The grid is a multiple of 8 with as many workgroups per XCD as
// an even range would hold work items, up to what its CUs hold.
hipError_t launch_sc2(const Work &w, int64_t items, int num_cus, hipStream_t s)
{
    const int mode = !w.learned ? kSc2Plain : w.feat_all ? kSc2Features : kSc2Learned;
    const int cus = std::max(1, num_cus / 8);
    const int grid = (int)(8 * std::min<int64_t>(4 * ((items + 7) / 8), cus * kSc2PerCu));
    if (mode == kSc2Plain) hipLaunchKernelGGL(k_sc2<kSc2Plain>, dim3(grid), dim3(256), sc2_lds(kSc2Plain), s, w);
    else if (mode == kSc2Learned) hipLaunchKernelGGL(k_sc2<kSc2Learned>, dim3(grid), dim3(256), sc2_lds(kSc2Learned), s, w);
    else hipLaunchKernelGGL(k_sc2<kSc2Features>, dim3(grid), dim3(256), sc2_lds(kSc2Features), s, w);
    return hipGetLastError();
}

hipError_t setup_graph_kernels()
{
    const void *fns[] = {reinterpret_cast<const void *>(k_sc2_sparse<kSc2Plain, false>),
                         reinterpret_cast<const void *>(k_sc2_sparse<kSc2Plain, true>),
                         reinterpret_cast<const void *>(k_sc2_sparse<kSc2Learned, false>),
                         reinterpret_cast<const void *>(k_sc2_sparse<kSc2Learned, true>),
                         reinterpret_cast<const void *>(k_sc2_sparse<kSc2Features, true>),
                         reinterpret_cast<const void *>(k_sc2<kSc2Learned>)};
    const int lds[] = {kSpLds, kSpLds, kSpLds, kSpLds, kSpLds, sc2_lds(kSc2Learned)};
    hipError_t e = hipSuccess;
    for (int k = 0; k < 6 && e == hipSuccess; ++k)
        e = hipFuncSetAttribute(fns[k], hipFuncAttributeMaxDynamicSharedMemorySize, lds[k]);
    return e;
}

}  // namespace tr
