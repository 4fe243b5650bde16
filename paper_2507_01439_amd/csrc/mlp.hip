// Learned pivot scorer on gfx950: per-match features, a 19 -> 64 -> 64 -> 1
// GELU MLP with bfloat16 weights and activations and float32 accumulation,
// the learned pivot reorder with plain SC2 order as fallback, and the
// training kernels (forward/backward with the weight gradients, reduction and Adam).
#include <algorithm>
#include <type_traits>
#include <vector>

#include "mlp.h"

namespace tr {
namespace {

constexpr float kGeluC = 0.7978845608028654f;   // sqrt(2/pi)

__device__ __forceinline__ uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);   // NaN stays NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ float bfround(float f) { return bf2f(f2bf(f)); }

// tanh-form GELU (Hendrycks & Gimpel 2016).
__device__ __forceinline__ float gelu(float x)
{
    return 0.5f * x * (1.0f + tanhf(kGeluC * (x + 0.044715f * x * x * x)));
}

// Parameters in LDS as float32: the weights are the bfloat16 copies, the biases the master values.
struct MlpLds {
    float p[TR_MLP_NPARAM];
};

__device__ void load_params(MlpLds &L, const uint16_t *wbf16, const float *w32)
{
    for (int k = threadIdx.x; k < TR_MLP_NPARAM; k += blockDim.x) {
        const bool bias = (k >= kB1 && k < kW2) || (k >= kB2 && k < kW3) || k == kB3;
        L.p[k] = bias ? w32[k] : bf2f(wbf16[k]);
    }
}

// Forward pass of one sample (inference): float32 accumulation, bfloat16
// activations. Layer 1 is fully unrolled so a1 stays in registers.
__device__ float forward(const MlpLds &L, const float (&x)[19])
{
    float a1[64];
#pragma unroll
    for (int o = 0; o < 64; ++o) {
        float acc = L.p[kB1 + o];
#pragma unroll
        for (int k = 0; k < 19; ++k) acc = __builtin_fmaf(L.p[kW1 + 19 * o + k], x[k], acc);
        a1[o] = bfround(gelu(acc));
    }
    float s = L.p[kB3];
#pragma unroll 2
    for (int o = 0; o < 64; ++o) {
        float acc = L.p[kB2 + o];
#pragma unroll
        for (int k = 0; k < 64; ++k) acc = __builtin_fmaf(L.p[kW2 + 64 * o + k], a1[k], acc);
        s = __builtin_fmaf(L.p[kW3 + o], bfround(gelu(acc)), s);
    }
    return s;
}

// ---------------------------------------------------------------- features

// Sum and maximum of row i of the SC2 matrix from the parts k, k + step, .. that the SC2 kernels left: the row's own
// segments and, the matrix being symmetric, its column's blocks above.
__device__ __forceinline__ void sc2_row_parts(const Work &w, const PairDesc &d, int i, int k, int step, int &sum, int &mx)
{
    const int64_t at = d.g_off / 64 + part_at(i, 0, d.npad / 64), ct = d.g_off / 128 + part_at(i, 0, d.npad / 128);
    sum = mx = 0;
#pragma unroll 4
    for (int s = i / 64 + k; s < (d.n + 63) / 64; s += step) {
        sum += w.rowsum[at + 32 * s];
        mx = max(mx, (int)w.segmax[at + 32 * s]);
    }
#pragma unroll 4
    for (int s = k; s <= i / 128; s += step) {
        sum += w.colsum[ct + 32 * s];
        mx = max(mx, (int)w.colmax[ct + 32 * s]);
    }
}

// 19 values per match from the integer accumulators (degree, 16-bin delta histogram)
// and the SC2 kernels' parts (row sum and maximum): ratios formed in float64, rounded to float32,
// then to bfloat16.
__global__ void __launch_bounds__(256) k_features(Work w, uint16_t *packed)
{
    const int total = stage_total(w, kPrep);
    for (int item = blockIdx.x; item < total; item += gridDim.x) {
        int local;
        const int b = stage_pair(w, kPrep, item, local);
        const PairDesc d = pair_desc(w, b);
        const int i = local * kPrepRows + threadIdx.x;
        if (i >= d.n) continue;
        const int32_t *rs = w.rowstat + ((int64_t)b * w.max_n + i) * 20;
        int sum, mx;
        sc2_row_parts(w, d, i, 0, 1, sum, mx);
        const double n1 = (double)(d.n - 1), n = (double)d.n;
        uint16_t *f = packed ? packed + (int64_t)(d.pt_off + i) * 19 : w.feat + ((int64_t)b * w.max_n + i) * 19;
        f[0] = f2bf((float)((double)rs[0] / n1));
        f[1] = f2bf((float)((double)sum / (n1 * n)));
        f[2] = f2bf((float)((double)mx / n));
#pragma unroll
        for (int k = 0; k < 16; ++k) f[3 + k] = f2bf((float)((double)rs[3 + k] / n1));
    }
}

// ---------------------------------------------------------------- inference + reorder

// Sum over the 64 lanes (DPP), valid in every lane.
__device__ __forceinline__ int wave_total(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2, 3
    return __builtin_amdgcn_readlane(v, 63);
}

// The scorer's weights in LDS, unit-minor so that lane o of a wave reads
// unit o's weight for input k from consecutive words (no bank conflicts); rows
// padded to 65 words so that the staging writes, which follow the parameters'
// global (unit-major) order, fall in distinct banks too.
struct MlpWave {
    static constexpr int kPad = 65;
    float w1[19][kPad], w2[64][kPad], b1[64], b2[64], w3[64], b3;
    // Thread tid's share of the weights (coalesced loads of the parameter
    // vector), fetched into registers early and written to LDS later (put), so
    // that the global reads overlap other work.
    struct Share {
        float a[5], c[16], e[3], f;
    };
    __device__ static Share fetch(const uint16_t *wbf16, const float *w32, int tid)
    {
        Share r;
#pragma unroll
        for (int u = 0; u < 5; ++u) r.a[u] = tid + 256 * u < 19 * 64 ? bf2f(wbf16[kW1 + tid + 256 * u]) : 0.0f;
#pragma unroll
        for (int u = 0; u < 16; ++u) r.c[u] = bf2f(wbf16[kW2 + tid + 256 * u]);
        const int t = tid & 63;
        r.e[0] = w32[kB1 + t];
        r.e[1] = w32[kB2 + t];
        r.e[2] = bf2f(wbf16[kW3 + t]);
        r.f = w32[kB3];
        return r;
    }
    // By a whole 256-thread workgroup; the caller synchronises after.
    __device__ void put(const Share &r, int tid)
    {
#pragma unroll
        for (int u = 0; u < 5; ++u) {
            const int t = tid + 256 * u;   // W1[o][k], o = t / 19, k = t % 19
            if (t < 19 * 64) w1[t % 19][t / 19] = r.a[u];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int t = tid + 256 * u;   // W2[o][k], o = t / 64, k = t % 64
            w2[t & 63][t >> 6] = r.c[u];
        }
        if (tid < 64) {
            b1[tid] = r.e[0];
            b2[tid] = r.e[1];
            w3[tid] = r.e[2];
        }
        if (tid == 0) b3 = r.f;
    }
    // Score of one match by a whole wave: lane o computes hidden unit o, each
    // layer one multiply-add chain per lane over inputs broadcast from the
    // wave's LDS row x (64 floats), in the same order as the one-thread forward
    // pass. fb: lane k < 19 holds feature k (bfloat16 bits).
    __device__ float score(uint16_t fb, int lane, float *x) const
    {
        auto publish = [&](float v) {   // every lane's value to x, visible to the whole wave
            x[lane] = v;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        };
        publish(lane < 19 ? bf2f(fb) : 0.0f);
        float acc = b1[lane];
#pragma unroll
        for (int k = 0; k < 19; ++k) acc = __builtin_fmaf(w1[k][lane], x[k], acc);
        const float a1 = bfround(gelu(acc));
        __builtin_amdgcn_wave_barrier();   // every lane has read the features
        publish(a1);
        acc = b2[lane];
#pragma unroll
        for (int k = 0; k < 64; ++k) acc = __builtin_fmaf(w2[k][lane], x[k], acc);
        const float a2 = bfround(gelu(acc));
        __builtin_amdgcn_wave_barrier();
        publish(a2);
        float s = b3;
#pragma unroll
        for (int o = 0; o < 64; ++o) s = __builtin_fmaf(w3[o], x[o], s);
        __builtin_amdgcn_wave_barrier();   // x is free for the wave's next row
        return s;
    }
};

// Feature k of a match from its integer accumulator v, as k_features.
__device__ __forceinline__ uint16_t feature_bits(int32_t v, int k, int n)
{
    const double n1 = (double)(n - 1), nn = (double)n;
    return f2bf((float)((double)v / (k == 0 ? n1 : k == 1 ? n1 * nn : k == 2 ? nn : n1)));
}

constexpr int kCandRows = 4;   // rows evaluated together against each loaded point

// Pool entry r moves to slot rk (kept if rk < K1); slots past the pair's K pivots are empty.
__device__ __forceinline__ void place_pivot(const Work &w, int b, int K, int p, uint64_t mine, int rk)
{
    const int32_t *pl = w.pivots_plain + (int64_t)b * w.pool_cap * 3;
    int32_t *out = w.pivots + (int64_t)b * w.piv_stride * 3;
    if (p < K && rk < w.k1) {
        const int r = (int)(uint32_t)mine;
        out[3 * rk] = pl[3 * r];
        out[3 * rk + 1] = pl[3 * r + 1];
        out[3 * rk + 2] = pl[3 * r + 2];
    }
    if (p >= K && p < w.k1) {
        out[3 * p] = -1;
        out[3 * p + 1] = -1;
        out[3 * p + 2] = 0;
    }
}

// Features and score of every match the reorder needs: the endpoints of the
// pair's plain pivot pool. The endpoints are cut into chunks of R (at most
// kCandRows); wave 0 claims each distinct row of its chunk by compare-and-swap
// on the row's mark, so every row is evaluated once. The workgroup then reads
// each of the pair's points once and evaluates delta_ij against all claimed
// rows, exactly as the compatibility kernel does (same operation order,
// correctly rounded square roots), counting the degree and the 16-bin delta
// histogram; the SC2 row sum and maximum are added up from the SC2 kernels'
// parts, a row per wave. Each wave then scores the rows
// of its slot. Matches outside the pool get no features and no score.
//
__global__ void __launch_bounds__(256, 2) k_cand_rows(Work w, int B, int R, const uint16_t *wbf16, const float *w32)
{
    __shared__ float crd[kCandRows][6];
    __shared__ int32_t row_l[kCandRows], rsv_l[kCandRows][2];
    __shared__ int32_t cnt_l;
    __shared__ int32_t red[4][kCandRows][9];
    __shared__ MlpWave mlp;
    __shared__ float act_l[4][64];   // per-wave broadcast row of the scorer
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    {   // the weights go to LDS while the first chunk's loads are in flight (first barrier below)
        const MlpWave::Share share = MlpWave::fetch(wbf16, w32, tid);
        mlp.put(share, tid);
    }
    const float tau = w.tau, q = tau * 0.25f;
    float edge[16];
#pragma unroll
    for (int k = 1; k < 16; ++k) edge[k] = (float)k * q;   // bin edges as the compatibility kernel forms them
    // Fast bin decision: t = delta / q in float32 is within 2^-22 t of the quotient and v_sqrt_f32
    // moves delta by at most 2^-21 (|x| + |y|); away from every edge by the guard band
    // 2^-19 (|x| + |y|) + 2e-6 + 2^-17 q, floor(t) is the bin and delta <= tau is decided.
    const float inv_q = 1.0f / q, guard0 = __builtin_fmaf(q, 0x1p-17f, 2e-6f);
    const int cpp = (2 * w.pool + R - 1) / R, total = B * cpp;
    for (int c = blockIdx.x; c < total; c += gridDim.x) {
        const int slot = c / cpp, b = batch_pair(w, slot), e0 = (c - slot * cpp) * R;
        const PairDesc d = pair_desc(w, b);
        if (e0 < 2 * d.kpiv) {   // the same for the whole workgroup
            // Two batches of kU points per thread are in flight before the rows are claimed
            // (N <= 4096 takes one round trip); later batches are fetched into the buffer
            // just consumed while the other one is evaluated.
            constexpr int kU = 8;
            float pa[kU][6], pb[kU][6];
            auto fetch_points = [&](float (&p)[kU][6], int j0) {
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const int64_t gj = d.pt_off + min(j0 + 256 * u, d.n - 1);
                    const float3 a = *reinterpret_cast<const float3 *>(w.src + 3 * gj);   // one 12-byte load
                    const float3 cc = *reinterpret_cast<const float3 *>(w.dst + 3 * gj);
                    p[u][0] = a.x; p[u][1] = a.y; p[u][2] = a.z;
                    p[u][3] = cc.x; p[u][4] = cc.y; p[u][5] = cc.z;
                }
            };
            fetch_points(pa, tid);
            if (256 * kU < d.n) fetch_points(pb, tid + 256 * kU);
            int pos = -1;   // wave 0: the lane's place among the claimed rows
            if (wv == 0) {
                const int e = e0 + lane;
                int i = -1;
                if (lane < R && e < 2 * d.kpiv) {
                    i = w.pivots_plain[((int64_t)b * w.pool_cap + (e >> 1)) * 3 + (e & 1)];
                    if (i < 0 || i >= d.n || atomicCAS(&w.mark[(int64_t)b * w.max_n + i], 0, 1) != 0) i = -1;
                }
                const uint64_t m = __ballot(i >= 0);
                if (i >= 0) {
                    pos = __popcll(m & ((1ull << lane) - 1ull));
                    const int64_t gi = d.pt_off + i;
                    row_l[pos] = i;
                    crd[pos][0] = w.src[3 * gi]; crd[pos][1] = w.src[3 * gi + 1]; crd[pos][2] = w.src[3 * gi + 2];
                    crd[pos][3] = w.dst[3 * gi]; crd[pos][4] = w.dst[3 * gi + 1]; crd[pos][5] = w.dst[3 * gi + 2];
                }
                if (lane == 0) cnt_l = __popcll(m);
            }
            __syncthreads();
            const int cnt = cnt_l;
            if (cnt > 0) {   // the same for the whole workgroup
                int rsum = 0, rmax = 0;   // wave r: the lane's parts of claimed row r's SC2 statistics
                if (wv < cnt) sc2_row_parts(w, d, __builtin_amdgcn_readfirstlane(row_l[wv]), lane, 64, rsum, rmax);
                uint32_t cw[kCandRows][4];   // 16 bins, 8 bits each (at most ceil(32767/256) per thread)
                int deg[kCandRows];
#pragma unroll
                for (int r = 0; r < kCandRows; ++r) {
                    deg[r] = 0;
                    cw[r][0] = cw[r][1] = cw[r][2] = cw[r][3] = 0;
                }
                auto eval_points = [&](float (&p)[kU][6], int j0) {
#pragma unroll
                    for (int u = 0; u < kU; ++u) {
                        const int j = j0 + 256 * u;
#pragma unroll
                        for (int r = 0; r < kCandRows; ++r) {
                            if (r >= cnt) break;
                            // hardware square roots first; a pair whose delta lies within the guard
                            // band of a bin edge k q (tau = 4 q is edge 4) is evaluated again with
                            // the correctly rounded ones, so every decision is the exact one
                            const float ax = crd[r][0] - p[u][0], ay = crd[r][1] - p[u][1], az = crd[r][2] - p[u][2];
                            const float bx = crd[r][3] - p[u][3], by = crd[r][4] - p[u][4], bz = crd[r][5] - p[u][5];
                            float s1 = ax * ax, s2 = bx * bx;
                            s1 = __builtin_fmaf(ay, ay, s1);
                            s2 = __builtin_fmaf(by, by, s2);
                            s1 = __builtin_fmaf(az, az, s1);
                            s2 = __builtin_fmaf(bz, bz, s2);
                            const float la = __builtin_amdgcn_sqrtf(s1), lb = __builtin_amdgcn_sqrtf(s2);
                            float dl = __builtin_fabsf(la - lb);
                            const float t = dl * inv_q;
                            const float kn = __builtin_fminf(__builtin_fmaxf(__builtin_rintf(t), 1.0f), 15.0f);
                            const float guard = __builtin_fmaf(la + lb, 0x1p-19f, guard0);
                            int bin;
                            if (__builtin_fabsf(dl - kn * q) <= guard || !(dl == dl)) {
                                const float lx = length32(ax, ay, az), ly = length32(bx, by, bz);
                                dl = __builtin_fabsf(lx - ly);
                                bin = 0;
#pragma unroll
                                for (int k = 1; k < 16; ++k) bin += dl >= edge[k];
                            } else {
                                bin = (int)__builtin_fminf(t, 15.0f);   // t >= 0, at least the guard from an integer
                            }
                            const bool in = j < d.n && j != row_l[r];
                            deg[r] += in && dl <= tau;
                            const uint32_t inc = in ? 1u << (8 * (bin & 3)) : 0u;
                            cw[r][0] += (bin >> 2) == 0 ? inc : 0u;
                            cw[r][1] += (bin >> 2) == 1 ? inc : 0u;
                            cw[r][2] += (bin >> 2) == 2 ? inc : 0u;
                            cw[r][3] += (bin >> 2) == 3 ? inc : 0u;
                        }
                    }
                };
                for (int j0 = tid; j0 < d.n; j0 += 2 * 256 * kU) {
                    eval_points(pa, j0);
                    if (j0 + 2 * 256 * kU < d.n) fetch_points(pa, j0 + 2 * 256 * kU);
                    if (j0 + 256 * kU < d.n) eval_points(pb, j0 + 256 * kU);
                    if (j0 + 3 * 256 * kU < d.n) fetch_points(pb, j0 + 3 * 256 * kU);
                }
                // Per row: bytes 0,2 and 1,3 of each counter word widen to 16-bit
                // fields (a workgroup's count of one bin is below 2^15).
#pragma unroll
                for (int r = 0; r < kCandRows; ++r) {
                    if (r >= cnt) break;
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const int te = wave_total((int)(cw[r][m] & 0x00FF00FFu));
                        const int to = wave_total((int)((cw[r][m] >> 8) & 0x00FF00FFu));
                        if (lane == 0) {
                            red[wv][r][2 * m] = te;
                            red[wv][r][2 * m + 1] = to;
                        }
                    }
                    const int td = wave_total(deg[r]);
                    if (lane == 0) red[wv][r][8] = td;
                }
                if (wv < cnt) {
                    rsum = wave_total(rsum);
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) rmax = max(rmax, __shfl_xor(rmax, o, 64));
                    if (lane == 0) {
                        rsv_l[wv][0] = rsum;
                        rsv_l[wv][1] = rmax;
                    }
                }
                __syncthreads();
#pragma unroll 1
                for (int r = wv; r < cnt; r += 4) {
                    const int i = row_l[r];
                    int32_t *rs = w.rowstat + ((int64_t)b * w.max_n + i) * 20;
                    int32_t v = 0;
                    if (lane == 0) {
                        v = red[0][r][8] + red[1][r][8] + red[2][r][8] + red[3][r][8];
                    } else if (lane < 3) {
                        v = rsv_l[r][lane - 1];   // SC2 row sum / maximum
                    } else if (lane < 19) {
                        const int bin = lane - 3, idx = 2 * (bin >> 2) + (bin & 1), sh = 16 * ((bin >> 1) & 1);
#pragma unroll
                        for (int g = 0; g < 4; ++g) v += (red[g][r][idx] >> sh) & 0xFFFF;
                    }
                    uint16_t fb = 0;
                    if (lane < 19) {
                        if (lane == 0 || lane >= 3) rs[lane] = v;
                        fb = feature_bits(v, lane, d.n);
                        w.feat[((int64_t)b * w.max_n + i) * 19 + lane] = fb;
                    }
                    const float sc = mlp.score(fb, lane, act_l[wv]);
                    if (lane == 0) {
                        w.scores[(int64_t)b * w.max_n + i] = sc;
                        if (!isfinite(sc)) atomicOr(&w.state[b].fallback, 1);
                    }
                }
            }
        }
        __syncthreads();   // row_l, crd, red, rsv_l and cnt_l are the next chunk's
    }
}

// Order the pool of plain pivots by e = s_i + s_j (desc), ties by plain rank,
// keep the first K1. Non-finite scores anywhere in the pair: keep plain order.
// Keys are distinct (the plain rank is part of each), so a key's new position
// is the number of smaller keys: each 256-thread workgroup rebuilds the
// pair's K keys in LDS and ranks 64 of them, a quarter of the list per wave,
// eight 16-byte broadcast reads in flight. (Pools larger than kFusedPool; the hypothesis
// kernel orders smaller ones.)
__global__ void __launch_bounds__(256) k_reorder(Work w, int blocks_per_pair)
{
    extern __shared__ uint64_t keys[];
    __shared__ int32_t part[4][64];
    const int slot = blockIdx.x / blocks_per_pair, b = batch_pair(w, slot), g = blockIdx.x - slot * blocks_per_pair;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const PairDesc d = pair_desc(w, b);
    const int K = d.kpiv;
    if (g * 64 >= max(K, w.k1)) return;
    const bool fb = w.state[b].fallback != 0;
    const int32_t *pl = w.pivots_plain + (int64_t)b * w.pool_cap * 3;
    const float *sc = w.scores + (int64_t)b * w.max_n;
    const int K16 = (K + 15) & ~15;
    for (int r = tid; r < K16; r += 256) keys[r] = r < K ? reorder_key(pl, sc, r, fb) : ~0ull;
    __syncthreads();
    const int p = g * 64 + lane;
    const uint64_t mine = p < K ? keys[p] : 0;
    const int per = ((K16 / 16 + 3) / 4) * 16;
    const int q0 = min(K16, wv * per), q1 = min(K16, q0 + per);
    part[wv][lane] = count_smaller(keys, q0, q1, mine);
    __syncthreads();
    if (wv != 0) return;
    const int rk = part[0][lane] + part[1][lane] + part[2][lane] + part[3][lane];
    place_pivot(w, b, K, p, mine, rk);
}

// ---------------------------------------------------------------- standalone forward

__global__ void __launch_bounds__(256) k_mlp_forward(const uint16_t *feat, int64_t m, float *scores,
                                                     const uint16_t *wbf16, const float *w32)
{
    __shared__ MlpLds L;
    load_params(L, wbf16, w32);
    __syncthreads();
    for (int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x; n < m; n += (int64_t)gridDim.x * 256) {
        float x[19];
#pragma unroll
        for (int k = 0; k < 19; ++k) x[k] = bf2f(feat[n * 19 + k]);
        scores[n] = forward(L, x);
    }
}

// ---------------------------------------------------------------- training

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));

// GELU and its derivative with one exponential and one reciprocal: with u = c (x + 0.044715 x^3),
// (1 + tanh u) / 2 = sigma(2u) = s, so gelu = x s and gelu' = s + x s (1 - s) 2 u'. No cancellation for
// negative x (1 + tanh u loses its digits there); the tanh form's call is some forty instructions. Far to the left
// 1 + exp(-2u) is infinite and s is 0 whatever the size of x (the Newton step alone works on a bounded one).
__device__ __forceinline__ void gelu_both(float x, float &a, float &g)
{
    constexpr float kL = -2.0f * kGeluC * 1.4426950408889634f;   // exp(-2u) = 2^(kL (x + 0.044715 x^3))
    const float x2 = x * x;
    const float p = 1.0f + __builtin_amdgcn_exp2f(x * __builtin_fmaf(0.044715f * kL, x2, kL));
    const float s0 = __builtin_amdgcn_rcpf(p);
    const float s = __builtin_fmaf(__builtin_fmaf(-fminf(p, 0x1p126f), s0, 1.0f), s0, s0);   // one Newton step
    a = x * s;
    g = __builtin_fmaf(__builtin_fmaf(-a, s, a), __builtin_fmaf(6.0f * 0.044715f * kGeluC, x2, 2.0f * kGeluC), s);
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)   // round to nearest even
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f{lo, hi}), v2bf));
}

__device__ __forceinline__ float lo_bf16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_bf16(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ __forceinline__ v16f mfma_bf16(v4u a, v4u b, v16f c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

// x and y as three bfloat16 terms each (8 + 8 + 8 bits: x = t[0] + t[1] + t[2] exactly, short of
// underflow), packed in pairs.
__device__ __forceinline__ void split3(float x, float y, uint32_t (&t)[3])
{
    const uint32_t xu = __float_as_uint(x), yu = __float_as_uint(y);
    t[0] = __builtin_amdgcn_perm(yu, xu, 0x07060302);
    const float x1 = x - __uint_as_float(xu & 0xFFFF0000u), y1 = y - __uint_as_float(yu & 0xFFFF0000u);
    const uint32_t x1u = __float_as_uint(x1), y1u = __float_as_uint(y1);
    t[1] = __builtin_amdgcn_perm(y1u, x1u, 0x07060302);
    const float x2 = x1 - __uint_as_float(x1u & 0xFFFF0000u), y2 = y1 - __uint_as_float(y1u & 0xFFFF0000u);
    t[2] = __builtin_amdgcn_perm(__float_as_uint(y2), __float_as_uint(x2), 0x07060302);
}

// Accumulator layout to operand layout: the eight packed words of a 32 x 32 block (word 2g + h: rows
// 8g + 4 lh + 2h, + 1 of the lane's column) become the two 16-row operands (lane: rows 16s + 8 lh .. + 7).
__device__ __forceinline__ void to_operand(uint32_t (&p)[8], v4u (&f)[2])
{
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const auto r = __builtin_amdgcn_permlane32_swap(p[4 * s + h], p[4 * s + 2 + h], false, false);
            f[s][h] = r[0];
            f[s][2 + h] = r[1];
        }
    }
}

__device__ __forceinline__ void wave_fence()   // LDS written by the wave's lanes is visible to all of them
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int kSamples = 32;    // samples per wave step
constexpr int kTPitch = 72;     // bfloat16 per LDS row of 64: 16-byte reads of eight rows fall in distinct banks
constexpr int kXPitch = 40;     // per LDS row of 32
constexpr int kTrainWaves = 4;  // waves per workgroup, one per SIMD
constexpr int kSums = 26;       // float4 a lane brings to the workgroup's sum

struct TrainWave {              // a wave's own LDS
    uint16_t t[3][kSamples * kTPitch];   // [sample][unit]: the features, layer 1's activations, the three
                                         // terms of layer 2's deltas, in turn
    uint16_t xt[32 * kXPitch];           // [feature][sample]; row 19 holds ones, rows 20 .. zeros
    float ds[kSamples];
};

struct TrainWeights {           // the workgroup's
    uint16_t w1[64 * kXPitch];  // [unit][feature]; columns 19-21 the bias as three bfloat16 terms, then zeros
    uint16_t w2[64 * kTPitch], w2t[64 * kTPitch];   // [out][in] and [in][out]
};

static_assert(kTrainWaves == 4, "the workgroup's sum adds four slots");
constexpr size_t kStepLds = sizeof(TrainWeights) + kTrainWaves * sizeof(TrainWave);
constexpr size_t kSumLds = (size_t)kTrainWaves * kSums * 64 * 16;
constexpr size_t kTrainLds = kStepLds > kSumLds ? kStepLds : kSumLds;

// Gradients (and loss) of the mean BCE-with-logits over m samples, one wave per 32 samples: forward,
// backward and the weight gradients in one pass, nothing per sample in memory. Each layer is a
// contraction on the matrix cores (v_mfma_f32_32x32x16_bf16, float32 sums). The weights, features and
// activations are bfloat16, so the forward products are exact; the deltas stay float32: each is split
// into three bfloat16 terms whose sum is the delta itself, and their three products run on the same
// instruction. Against float64 (samples whose activations round alike on both sides) the gradients are off by 5e-8
// to 8e-8 relative at m = 1000 .. 200000, the float32 multiply-adds' by 8e-8 to 3.5e-7.
//
// Accumulators hold one unit per lane and 16 of the samples, (lane: unit l31 of a 32-block; entry r:
// sample 8 (r / 4) + 4 lh + r % 4). With deltas and activations in that layout the weight gradients
// (contractions over the samples) take their operands by exchanges between the wave's halves alone; the
// two products over units (layer 2 forward, and back to layer 1) read them as [sample][unit] from the
// wave's LDS. Ones beside the features make the layer-1 bias (three bfloat16 terms) and its gradient
// columns of the same products.
//
// Waves step through the samples with their gradient sums in registers; the workgroup adds its waves'
// sums pairwise through LDS and writes one partial, and k_mlp_reduce adds the partials, all in a fixed
// order. At m = 65536 this and the reduction take 26.2 + 4.5 us, at m = 2125 16.4 + 4.0 (a thread per sample
// with the activations and deltas in memory, weight gradients by a second kernel: 111.5 + 35.5 + 13.3 and
// 92.6 + 30.1 + 4.7). What bounds it is vector issue (64 GELUs, their gradients and the splits per lane and
// step) with one wave per SIMD: two waves per SIMD need at most 256 registers and spilled 230 (65 us).
__global__ void __launch_bounds__(64 * kTrainWaves) k_mlp_train(const uint16_t *feat, const uint8_t *labels, int64_t m,
                                                       const uint16_t *wbf16, const float *w32, float *partial)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    TrainWeights &W = *reinterpret_cast<TrainWeights *>(smem);
    const int tid = threadIdx.x, lane = tid & 63, l31 = lane & 31, lh = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    TrainWave &L = *reinterpret_cast<TrainWave *>(smem + sizeof(TrainWeights) + wv * sizeof(TrainWave));
    const int64_t tiles = (m + kSamples - 1) / kSamples, stride = (int64_t)gridDim.x * kTrainWaves;
    int64_t tile = (int64_t)blockIdx.x * kTrainWaves + wv;
    const float inv_m = 1.0f / (float)m;
    // a step's features, fetched ahead: lane's sample xn, features xk .. xk + 9 (two-byte loads: a slice of a
    // feature table need not be aligned further)
    const int xn = lane >> 1, xk = 10 * (lane & 1);
    uint16_t xv[10];
    auto fetch = [&](int64_t t) {
        const bool ok = t * kSamples + xn < m;
        const uint16_t *f = feat + (t * kSamples + xn) * 19 + xk;
#pragma unroll
        for (int u = 0; u < 10; ++u) xv[u] = ok && xk + u < 19 ? f[u] : 0;
    };
    fetch(tile);
    // ---- weights
    for (int k = tid; k < 64 * kXPitch; k += 64 * kTrainWaves) {
        const int o = k / kXPitch, c = k % kXPitch;
        uint16_t v = 0;
        if (c < 19) v = wbf16[kW1 + 19 * o + c];
        else if (c < 22) {
            uint32_t t[3];
            split3(w32[kB1 + o], 0.0f, t);
            v = (uint16_t)t[c - 19];
        }
        W.w1[k] = v;
    }
    for (int k = tid; k < 64 * 8; k += 64 * kTrainWaves) {
        const int o = k >> 3, c = 8 * (k & 7);
        const uint4 v = *reinterpret_cast<const uint4 *>(wbf16 + kW2 + 64 * o + c);
        *reinterpret_cast<uint4 *>(&W.w2[o * kTPitch + c]) = v;
        const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) W.w2t[(c + e) * kTPitch + o] = (uint16_t)(u[e >> 1] >> (16 * (e & 1)));
    }
    float w3[2], b2[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        w3[b] = bf2f(wbf16[kW3 + 32 * b + l31]);
        b2[b] = w32[kB2 + 32 * b + l31];
    }
    const float b3 = w32[kB3];
    for (int k = lane; k < 13 * 32; k += 64) L.xt[(19 + (k >> 5)) * kXPitch + (k & 31)] = k < 32 ? 0x3F80 : 0;
    __syncthreads();
    auto frag = [&](const uint16_t *t, int pitch, int row, int s) {   // columns 16s + 8 lh .. + 7 of a row
        return *reinterpret_cast<const v4u *>(&t[row * pitch + 16 * s + 8 * lh]);
    };
    v16f dw2[2][2] = {}, dw1[2] = {};
    float db2[2] = {0, 0}, dw3[2] = {0, 0}, db3 = 0.0f, loss = 0.0f;
    // this lane's sample after the logits' reduction over units (lanes 2k, 2k + 1 hold the same one)
    const int mr = l31 >> 1, ms = 8 * (mr >> 2) + 4 * lh + (mr & 3);
    for (; tile < tiles; tile += stride) {
        const int64_t n0 = tile * kSamples;
        const bool live = n0 + ms < m;
        const float y = live && labels[n0 + ms] ? 1.0f : 0.0f;
        // ---- features to LDS
        uint16_t *X = L.t[0];
#pragma unroll
        for (int u = 0; u < 10; ++u) {
            if (u < 9 || xk == 0) {
                X[xn * kXPitch + xk + u] = xv[u];
                L.xt[(xk + u) * kXPitch + xn] = xv[u];
            }
        }
        if (lane < 32) {   // the ones beside the features, zeros behind
            X[lane * kXPitch + 19] = 0x3F80;
            *reinterpret_cast<uint2 *>(&X[lane * kXPitch + 20]) = make_uint2(0x3F803F80u, 0u);
            *reinterpret_cast<uint4 *>(&X[lane * kXPitch + 24]) = make_uint4(0, 0, 0, 0);
        }
        wave_fence();
        if (tile + stride < tiles) fetch(tile + stride);
        // ---- layer 1: z1[n][o], a1 = bf16(gelu(z1)) packed by sample pairs, g1 = gelu'(z1)
        float g1[2][16];
        uint32_t a1[2][8];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            v16f z = {};
#pragma unroll
            for (int s = 0; s < 2; ++s) z = mfma_bf16(frag(X, kXPitch, l31, s), frag(W.w1, kXPitch, 32 * b + l31, s), z);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                float p, q;
                gelu_both(z[2 * k], p, g1[b][2 * k]);
                gelu_both(z[2 * k + 1], q, g1[b][2 * k + 1]);
                a1[b][k] = pack_bf16(p, q);
            }
        }
        // entry pair k of a lane: samples 8 (k / 2) + 4 lh + 2 (k % 2), + 1
        auto put = [&](uint16_t *t, int b, const uint32_t (&p)[8]) {   // to [sample][unit]
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                uint16_t *o = &t[(8 * (k >> 1) + 4 * lh + 2 * (k & 1)) * kTPitch + 32 * b + l31];
                o[0] = (uint16_t)p[k];
                o[kTPitch] = (uint16_t)(p[k] >> 16);
            }
        };
        v4u fa[2][2];   // a1 as the operand of dW2
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            put(L.t[1], b, a1[b]);
            to_operand(a1[b], fa[b]);
        }
        wave_fence();
        // ---- layer 2 and the logit
        float g2[2][16];
        uint32_t a2[2][8];
        {
            v16f z[2];
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) z[b][r] = b2[b];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const v4u a = frag(L.t[1], kTPitch, l31, s);
#pragma unroll
                for (int b = 0; b < 2; ++b) z[b] = mfma_bf16(a, frag(W.w2, kTPitch, 32 * b + l31, s), z[b]);
            }
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    float p, q;
                    gelu_both(z[b][2 * k], p, g2[b][2 * k]);
                    gelu_both(z[b][2 * k + 1], q, g2[b][2 * k + 1]);
                    a2[b][k] = pack_bf16(p, q);
                }
        }
        float pr[16];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            pr[2 * k] = __builtin_fmaf(w3[1], lo_bf16(a2[1][k]), w3[0] * lo_bf16(a2[0][k]));
            pr[2 * k + 1] = __builtin_fmaf(w3[1], hi_bf16(a2[1][k]), w3[0] * hi_bf16(a2[0][k]));
        }
        // sums over the 32 units, halving the samples a lane holds at each exchange: lane l31 ends with
        // sample entry l31 / 2
        auto fold = [&](auto cnt, auto xo) {
            constexpr int c = decltype(cnt)::value, x = decltype(xo)::value;
            const bool up = l31 & x;
#pragma unroll
            for (int k = 0; k < c; ++k) {
                const float keep = up ? pr[c + k] : pr[k], send = up ? pr[k] : pr[c + k];
                pr[k] = keep + __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(send), (x << 10) | 0x1f));
            }
        };
        fold(std::integral_constant<int, 8>{}, std::integral_constant<int, 16>{});
        fold(std::integral_constant<int, 4>{}, std::integral_constant<int, 8>{});
        fold(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
        fold(std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{});
        const float s = b3 + (pr[0] + __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(pr[0]), (1 << 10) | 0x1f)));
        const float ds_n = live ? (1.0f / (1.0f + expf(-s)) - y) * inv_m : 0.0f;
        if (!(lane & 1)) {
            L.ds[ms] = ds_n;
            db3 += ds_n;
            if (live) loss += (fmaxf(s, 0.0f) - s * y + log1pf(expf(-fabsf(s)))) * inv_m;
        }
        wave_fence();
        float ds[16];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 v = *reinterpret_cast<const float4 *>(&L.ds[8 * g + 4 * lh]);
            ds[4 * g] = v.x; ds[4 * g + 1] = v.y; ds[4 * g + 2] = v.z; ds[4 * g + 3] = v.w;
        }
        // ---- layer 2's deltas d2 = ds w3 gelu'(z2) in three terms; dW3, db2, dW2 = d2^T a1
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            uint32_t p[3][8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                dw3[b] = __builtin_fmaf(ds[2 * k], lo_bf16(a2[b][k]), dw3[b]);
                dw3[b] = __builtin_fmaf(ds[2 * k + 1], hi_bf16(a2[b][k]), dw3[b]);
                const float x = ds[2 * k] * w3[b] * g2[b][2 * k], z = ds[2 * k + 1] * w3[b] * g2[b][2 * k + 1];
                db2[b] += x;
                db2[b] += z;
                uint32_t t[3];
                split3(x, z, t);
                p[0][k] = t[0];
                p[1][k] = t[1];
                p[2][k] = t[2];
            }
#pragma unroll
            for (int q = 2; q >= 0; --q) {
                put(L.t[q], b, p[q]);
                v4u f[2];
                to_operand(p[q], f);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb) dw2[b][kb] = mfma_bf16(f[h], fa[kb][h], dw2[b][kb]);
            }
        }
        wave_fence();
        // ---- back to layer 1: d1 = (d2 W2) gelu'(z1); dW1 (and db1) = d1^T x
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            v16f z = {};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const v4u wf = frag(W.w2t, kTPitch, 32 * kb + l31, t);
#pragma unroll
                for (int q = 2; q >= 0; --q) z = mfma_bf16(frag(L.t[q], kTPitch, l31, t), wf, z);
            }
            uint32_t p[3][8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                uint32_t t[3];
                split3(z[2 * k] * g1[kb][2 * k], z[2 * k + 1] * g1[kb][2 * k + 1], t);
                p[0][k] = t[0];
                p[1][k] = t[1];
                p[2][k] = t[2];
            }
#pragma unroll
            for (int q = 2; q >= 0; --q) {
                v4u f[2];
                to_operand(p[q], f);
#pragma unroll
                for (int h = 0; h < 2; ++h) dw1[kb] = mfma_bf16(f[h], frag(L.xt, kXPitch, l31, h), dw1[kb]);
            }
        }
        wave_fence();   // the wave's LDS is the next step's
    }
    // ---- the workgroup's sum: the waves' sums in LDS, then each thread adds its entries and writes the partial
    float4 *slots = reinterpret_cast<float4 *>(smem);
    auto give = [&]() {
        float4 *o = slots + wv * kSums * 64 + lane;
        auto four = [&](int at, float a, float b, float c, float d) { o[at * 64] = make_float4(a, b, c, d); };
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    four(8 * b + 4 * kb + g, dw2[b][kb][4 * g], dw2[b][kb][4 * g + 1], dw2[b][kb][4 * g + 2],
                         dw2[b][kb][4 * g + 3]);
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                four(16 + 4 * b + g, dw1[b][4 * g], dw1[b][4 * g + 1], dw1[b][4 * g + 2], dw1[b][4 * g + 3]);
        four(24, db2[0], db2[1], dw3[0], dw3[1]);
        four(25, db3, loss, 0.0f, 0.0f);
    };
    __syncthreads();   // the steps' LDS is free
    give();
    __syncthreads();
    auto total = [&](int e) {
        const float4 a = slots[e], b = slots[e + kSums * 64], c = slots[e + 2 * kSums * 64], d = slots[e + 3 * kSums * 64];
        return make_float4((a.x + b.x) + (c.x + d.x), (a.y + b.y) + (c.y + d.y), (a.z + b.z) + (c.z + d.z),
                           (a.w + b.w) + (c.w + d.w));
    };
    float *out = partial + (int64_t)blockIdx.x * kGradSlots;
    for (int at = wv; at < 24; at += kTrainWaves) {   // rows o .. o + 3 of a weight gradient
        const float4 v = total(at * 64 + lane);
        const float e[4] = {v.x, v.y, v.z, v.w};
        const int b = at < 16 ? at >> 3 : (at >> 2) & 1, o = 32 * b + 8 * (at & 3) + 4 * lh, k = 32 * ((at >> 2) & 1) + l31;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (at < 16) out[kW2 + 64 * (o + j) + k] = e[j];
            else if (l31 < 19) out[kW1 + 19 * (o + j) + l31] = e[j];
            else if (l31 == 19) out[kB1 + o + j] = e[j];
        }
    }
    if (wv == 0 && !lh) {   // a unit's two halves of the samples
        const float4 v = total(24 * 64 + lane), u = total(24 * 64 + 32 + lane);
        out[kB2 + lane] = v.x + u.x;
        out[kB2 + 32 + lane] = v.y + u.y;
        out[kW3 + lane] = v.z + u.z;
        out[kW3 + 32 + lane] = v.w + u.w;
    }
    if (wv == 1) {
        float4 v = total(25 * 64 + lane);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            v.x += __shfl_xor(v.x, o, 64);
            v.y += __shfl_xor(v.y, o, 64);
        }
        if (lane == 0) {
            out[kB3] = v.x;
            out[TR_MLP_NPARAM] = v.y;
        }
    }
}

// Adam's step for one parameter (float32 master weight, bfloat16 copy).
struct AdamArgs {
    float *w, *mo, *ve;
    uint16_t *wbf16;
    float lr, c1, c2;
};

// Sum of the workgroups' partials per gradient slot, in a fixed order: four quarters of the list in
// order, then the quarters; kReduceBatch loads are issued together. With ADAM the parameter is
// updated at once.
constexpr int kReduceBatch = 32;
template <bool ADAM>
__global__ void __launch_bounds__(256) k_mlp_reduce(const float *partial, int parts, float *grads, float *loss,
                                                    AdamArgs ad)
{
    __shared__ float quarter[4][64];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6, p = blockIdx.x * 64 + lane;
    const int per = (parts + 3) / 4, t0 = q * per, t1 = min(parts, t0 + per);
    float acc = 0.0f;
    for (int t = t0; t < t1; t += kReduceBatch) {
        float v[kReduceBatch];
#pragma unroll
        for (int u = 0; u < kReduceBatch; ++u)
            v[u] = t + u < t1 && p < kGradSlots ? partial[(int64_t)(t + u) * kGradSlots + p] : 0.0f;
#pragma unroll
        for (int u = 0; u < kReduceBatch; ++u) acc += v[u];
    }
    quarter[q][lane] = acc;
    __syncthreads();
    if (q != 0 || p >= kGradSlots) return;
    const float g = (quarter[0][lane] + quarter[1][lane]) + (quarter[2][lane] + quarter[3][lane]);
    if (p == TR_MLP_NPARAM) {
        if (loss) *loss = g;
        return;
    }
    grads[p] = g;
    if (ADAM) {
        const float m = 0.9f * ad.mo[p] + 0.1f * g;
        const float v = 0.999f * ad.ve[p] + 0.001f * g * g;
        ad.mo[p] = m;
        ad.ve[p] = v;
        const float nw = ad.w[p] - ad.lr * (m / ad.c1) / (sqrtf(v / ad.c2) + 1e-8f);
        ad.w[p] = nw;
        ad.wbf16[p] = f2bf(nw);
    }
}

__global__ void k_to_bf16(const float *w, uint16_t *wbf16, int n)
{
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p < n) wbf16[p] = f2bf(w[p]);
}

int grid_for(int64_t m)
{
    const int64_t g = (m + 255) / 256;
    return (int)(g < 4096 ? (g > 0 ? g : 1) : 4096);
}

}  // namespace

hipError_t setup_mlp_kernels()
{
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_reorder),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, TR_MAX_POOL * (int)sizeof(uint64_t));
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_mlp_train), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)kTrainLds);
    return e;
}

hipError_t mlp_create(MlpState *s)
{
    hipError_t e = hipMalloc(&s->w32, sizeof(float) * TR_MLP_NPARAM);
    if (e == hipSuccess) e = hipMalloc(&s->m, sizeof(float) * TR_MLP_NPARAM);
    if (e == hipSuccess) e = hipMalloc(&s->v, sizeof(float) * TR_MLP_NPARAM);
    if (e == hipSuccess) e = hipMalloc(&s->wbf16, sizeof(uint16_t) * TR_MLP_NPARAM);
    if (e == hipSuccess) e = hipMalloc(&s->grads, sizeof(float) * kGradSlots);
    int device = 0, cus = 0;
    if (e == hipSuccess) e = hipGetDevice(&device);
    if (e == hipSuccess && hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && cus > 0)
        s->num_cus = cus;
    if (e == hipSuccess) e = hipMalloc(&s->partial, sizeof(float) * kGradSlots * (size_t)s->num_cus);
    return e;
}

void mlp_release(MlpState *s)
{
    for (void *p : {(void *)s->w32, (void *)s->m, (void *)s->v, (void *)s->wbf16, (void *)s->grads,
                    (void *)s->partial})
        if (p) hipFree(p);
    *s = MlpState();
}

hipError_t mlp_set(MlpState *s, const float *host)
{
    std::vector<float> zero(TR_MLP_NPARAM, 0.0f);
    hipError_t e = hipMemcpy(s->w32, host, sizeof(float) * TR_MLP_NPARAM, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(s->m, zero.data(), sizeof(float) * TR_MLP_NPARAM, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(s->v, zero.data(), sizeof(float) * TR_MLP_NPARAM, hipMemcpyHostToDevice);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_to_bf16, dim3((TR_MLP_NPARAM + 255) / 256), dim3(256), 0, 0, s->w32, s->wbf16, TR_MLP_NPARAM);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipDeviceSynchronize();
    s->step = 0;
    return e;
}

hipError_t mlp_get(MlpState *s, float *host)
{
    hipError_t e = hipDeviceSynchronize();
    if (e != hipSuccess) return e;
    return hipMemcpy(host, s->w32, sizeof(float) * TR_MLP_NPARAM, hipMemcpyDeviceToHost);
}

hipError_t mlp_forward(MlpState *s, const uint16_t *feat, int64_t m, float *scores, hipStream_t st)
{
    if (m == 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_forward, dim3(grid_for(m)), dim3(256), 0, st, feat, m, scores, s->wbf16, s->w32);
    return hipGetLastError();
}

namespace {

// Partials of the gradients over m samples, one per workgroup (*parts of them, at most one per CU).
hipError_t launch_train(MlpState *s, const uint16_t *feat, const uint8_t *labels, int64_t m, int *parts, hipStream_t st)
{
    const int64_t tiles = (m + kSamples - 1) / kSamples;
    *parts = (int)std::min<int64_t>((tiles + kTrainWaves - 1) / kTrainWaves, s->num_cus);
    hipLaunchKernelGGL(k_mlp_train, dim3(*parts), dim3(64 * kTrainWaves), kTrainLds, st, feat, labels, m, s->wbf16, s->w32,
                       s->partial);
    return hipGetLastError();
}

}  // namespace

hipError_t mlp_grads(MlpState *s, const uint16_t *feat, const uint8_t *labels, int64_t m, float *grads, float *loss,
                     hipStream_t st)
{
    int parts = 0;
    const hipError_t e = launch_train(s, feat, labels, m, &parts, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mlp_reduce<false>, dim3((kGradSlots + 63) / 64), dim3(256), 0, st, s->partial, parts, grads, loss,
                       AdamArgs{});
    return hipGetLastError();
}

hipError_t mlp_train_step(MlpState *s, const uint16_t *feat, const uint8_t *labels, int64_t m, float lr, float *loss,
                          hipStream_t st)
{
    int parts = 0;
    const hipError_t e = launch_train(s, feat, labels, m, &parts, st);
    if (e != hipSuccess) return e;
    s->step += 1;
    // bias corrections 1 - beta^t in float64: in float32, 1 - 0.999^t loses ~3e-5 relative to
    // cancellation at small t, which would move every early step by as much
    const float c1 = (float)(1.0 - pow(0.9, (double)s->step)), c2 = (float)(1.0 - pow(0.999, (double)s->step));
    hipLaunchKernelGGL(k_mlp_reduce<true>, dim3((kGradSlots + 63) / 64), dim3(256), 0, st, s->partial, parts, s->grads,
                       loss, AdamArgs{s->w32, s->m, s->v, s->wbf16, lr, c1, c2});
    return hipGetLastError();
}

hipError_t launch_features(const Work &w, uint16_t *packed, int grid, hipStream_t st)
{
    hipLaunchKernelGGL(k_features, dim3(grid), dim3(256), 0, st, w, packed);
    return hipGetLastError();
}

hipError_t launch_learned_order(const Work &w, const MlpState &mlp, int B, int grid, hipStream_t st)
{
    // Rows per chunk: few enough chunks that all run at once (two workgroups
    // per CU fit), at most kCandRows rows each.
    const int cand = B * 2 * w.pool;
    const int R = max(1, min(kCandRows, (cand + 2 * grid - 1) / (2 * grid)));
    const int chunks = B * ((2 * w.pool + R - 1) / R);
    hipLaunchKernelGGL(k_cand_rows, dim3(min(chunks, grid * 2)), dim3(256), 0, st, w, B, R, mlp.wbf16, mlp.w32);
    if (!w.rank_in_hyp) {   // small pools are ordered by the hypothesis kernel itself
        const int bpp = (max(w.pool, w.k1) + 63) / 64;
        hipLaunchKernelGGL(k_reorder, dim3(B * bpp), dim3(256), (size_t)((w.pool + 15) & ~15) * sizeof(uint64_t), st,
                           w, bpp);
    }
    return hipGetLastError();
}

}  // namespace tr
