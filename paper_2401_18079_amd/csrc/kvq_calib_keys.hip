// Offline per-channel calibration of the Keys (paper Sec. 3.6 and the appendix on offline calibration):
// per channel the k smallest and the k largest of the T calibration values are its outliers; thresholds
// are the k-th smallest / largest value, and the values strictly inside give the zero-point (mid-range)
// and scale (half-range).  With the channel's values sorted these are four order statistics: the k-th
// and the (k+1)-th from either end.
//
// Design (gfx950).  The matrix is [T][D], a channel a column of it.  Long calls that come with scratch memory read it once
// (second half of this file).  Without scratch memory a workgroup owns a group of neighbouring channels from the first row to the last: a load
// takes up to eight channels (16 bytes) of a row, two such lanes cover 16 channels.  Bound: HBM, two
// sweeps over the matrix.  Sweep one counts the high bytes of the order-preserving 16-bit keys (a
// 256-bin LDS histogram per channel), sweep two the low bytes inside the (at most four) bins that hold
// the order statistics.  Of many rows only the tails are counted: a sixteenth of the rows, counted in full first,
// bounds the order statistics (the K-th largest of any subset is at most the K-th largest of all), and
// keys inside the bounds skip the LDS atomics, which otherwise serialize on the few bins that hold the
// bulk of a channel.  Groups that read the same 128-byte lines are dispatched to one XCD (workgroup b
// runs on XCD b mod 8), so its L2 serves all but the first of them.
// Measured on 32768 x 4096: 182 us (one workgroup per channel with the column in LDS, each 2-byte element
// a line of its own: 1459 us).  With the arithmetic and the atomics taken out it takes 172 us: two sweeps
// of 32-byte row pieces at 3.2 TB/s.  Neighbouring groups spread over the XCDs: 326 us.  Eight loads in
// flight per thread instead of four, or the second sweep from the last row to the first: no change.
#include <math.h>
#include <type_traits>
#include "kvq_select.hpp"

namespace {

constexpr int CK_NT = 1024;
constexpr int CK_STRIDE = 16;            // every CK_STRIDE-th row is counted for the bounds
// sampled rows below which the sample is not worth its pass and its barriers (us with / without: 1024 rows of 256
// channels 10.9 / 9.9, 2048 rows of 5120 channels 31.8 / 29.2, 4096 rows of 4096 channels 24.5 / 24.0)
constexpr int CK_MIN_SAMPLE = 512;

// V consecutive fp16 values as raw dwords (V = 1: one value in the low half).
template <int V>
struct CkVec {
    uint32_t w[V < 2 ? 1 : V / 2];
};
template <int V>
__device__ __forceinline__ CkVec<V> ck_load(const uint16_t *p)
{
    CkVec<V> r;
    if constexpr (V == 8) {
        const uint4 v = *(const uint4 *)p;
        r.w[0] = v.x; r.w[1] = v.y; r.w[2] = v.z; r.w[3] = v.w;
    } else if constexpr (V == 4) {
        const uint2 v = *(const uint2 *)p;
        r.w[0] = v.x; r.w[1] = v.y;
    } else if constexpr (V == 2) {
        r.w[0] = *(const uint32_t *)p;
    } else {
        r.w[0] = *p;
    }
    return r;
}
// Two order-preserving keys at once.  -0 (key 0x7FFF) stays next to +0 (0x8000) here; the results map
// it to +0, which changes no value's rank among different values.
__device__ __forceinline__ uint32_t ck_keys(uint32_t two)
{
    typedef short s16x2 __attribute__((ext_vector_type(2)));
    const s16x2 x = __builtin_bit_cast(s16x2, two);
    const uint32_t sign = __builtin_bit_cast(uint32_t, x >> (short)15);
    return two ^ (sign | 0x80008000u);
}
__device__ __forceinline__ float ck_value(uint32_t key, uint16_t &bits)
{
    if (key == 0x7FFFu) key = 0x8000u;
    bits = (uint16_t)((key & 0x8000u) ? (key & 0x7FFFu) : (~key & 0xFFFFu));
    return kvq_h2f(bits);
}

// Calls f(row element index e, key) for the V values of every `step`-th row of this thread's rows.
template <int V, int LPR, class F>
__device__ __forceinline__ void ck_sweep(const uint16_t *__restrict__ col, int D, int T, int step, int row0, F f)
{
    constexpr int RPI = CK_NT / LPR;       // rows per workgroup step
    constexpr int U = 4;                   // loads in flight per thread
    const int n = (T + step - 1) / step;   // rows of the sweep
    for (int i0 = row0; i0 < n; i0 += RPI * U) {
        CkVec<V> v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * RPI;
            v[u] = ck_load<V>(col + (int64_t)(i < n ? i : i0) * step * D);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i0 + u * RPI < n) {
#pragma unroll
                for (int w = 0; w < (V < 2 ? 1 : V / 2); ++w) {
                    const uint32_t two = ck_keys(v[u].w[w]);
                    f(2 * w, two & 0xFFFFu);
                    if (V > 1) f(2 * w + 1, two >> 16);
                }
            }
        }
    }
}

// The constants of channel c from its order statistics' keys: k-th largest, (k+1)-th largest, k-th smallest, (k+1)-th smallest.
struct CkOut {
    uint16_t *s, *z, *lo, *hi;
};
__device__ __forceinline__ void ck_store(const CkOut &out, int c, int k, const uint32_t (&key)[4])
{
    uint16_t hb, lob, unused;
    const float a = ck_value(key[3], unused), b = ck_value(key[1], unused);
    ck_value(key[0], hb);
    ck_value(key[2], lob);
    const uint16_t zc = kvq_f2h_rn((b + a) * 0.5f);
    uint16_t sc = kvq_f2h_rn((b - a) * 0.5f);
    if (!(kvq_h2f(sc) > 0.0f)) sc = 0x3C00u;                      // 1.0
    out.s[c] = sc;
    out.z[c] = zc;
    out.lo[c] = (k > 0) ? lob : (uint16_t)0xFBFFu;                // -65504
    out.hi[c] = (k > 0) ? hb : (uint16_t)0x7BFFu;                 // +65504
}

// LPR lanes of V channels each: a workgroup owns C = V * LPR channels, group g of them.
template <int V, int LPR>
struct CkLds {
    // [C][4][256]: low-byte counts; the high-byte counts of sweep one are the same memory's first quarter
    __attribute__((aligned(16))) uint32_t cnt[V * LPR * 4 * 256];
    uint32_t bound[V * LPR];          // (first counted upper bin) << 8 | (last counted lower bin)
    uint32_t target[V * LPR];         // bins of the order statistics: top k, top k+1, bottom k, bottom k+1
};
template <int V, int LPR>
__device__ __forceinline__ void ck_two_sweeps(const uint16_t *__restrict__ k_cal, int T, int D, int k, int g,
                                              CkLds<V, LPR> &lds, const CkOut &out)
{
    constexpr int C = V * LPR;
    static_assert(C <= CK_NT / 64, "a wavefront per channel finds its bins");
    uint32_t *cnt = lds.cnt, *bound = lds.bound, *target = lds.target;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = tid % LPR, row0 = tid / LPR;
    const uint16_t *col = k_cal + (int64_t)g * C + lr * V;
    uint32_t *mine = cnt + lr * V * 256;   // sweep one: this lane's V histograms
    const uint32_t K1 = (uint32_t)k + 1u;

    for (int i = tid; i < C * 256; i += CK_NT) cnt[i] = 0;
    if (tid < C) bound[tid] = 0x00FFu;     // every bin
    __syncthreads();
    const int n_sample = (T + CK_STRIDE - 1) / CK_STRIDE;
    if (n_sample >= CK_MIN_SAMPLE && 2 * K1 <= (uint32_t)n_sample) {
        ck_sweep<V, LPR>(col, D, T, CK_STRIDE, row0,
                         [&](int e, uint32_t key) { atomicAdd(&mine[e * 256 + (key >> 8)], 1u); });
        __syncthreads();
        if (wave < C) {
            uint32_t top, bot, beyond, in_bin;
            wave_find_bin<true>(cnt + wave * 256, K1, lane, top, beyond, in_bin);
            wave_find_bin<false>(cnt + wave * 256, K1, lane, bot, beyond, in_bin);
            if (lane == 0) bound[wave] = (top << 8) | bot;
        }
        __syncthreads();
        for (int i = tid; i < C * 256; i += CK_NT) cnt[i] = 0;
        __syncthreads();
    }
    // bins strictly between the bounds are not counted: (bin - first) as unsigned is below `span` there
    uint32_t first[V], span[V];
    auto set_range = [&](int e, uint32_t upper, uint32_t lower) {
        first[e] = lower + 1u;
        span[e] = upper > lower + 1u ? upper - lower - 1u : 0u;
    };
#pragma unroll
    for (int e = 0; e < V; ++e) set_range(e, bound[lr * V + e] >> 8, bound[lr * V + e] & 255u);
    ck_sweep<V, LPR>(col, D, T, 1, row0, [&](int e, uint32_t key) {
        const uint32_t bin = key >> 8;
        if (bin - first[e] >= span[e]) atomicAdd(&mine[e * 256 + bin], 1u);
    });
    __syncthreads();
    // wavefront w looks after channel w: bins of the k-th and (k+1)-th from the top and from the bottom, and
    // how many elements lie beyond each
    uint32_t bin[4] = {0, 0, 0, 0}, beyond[4] = {0, 0, 0, 0};
    if (wave < C) {
        const uint32_t *h = cnt + wave * 256;
        uint32_t in_bin;
        wave_find_bin<true>(h, K1, lane, bin[1], beyond[1], in_bin);
        wave_find_bin<false>(h, K1, lane, bin[3], beyond[3], in_bin);
        bin[0] = bin[1]; beyond[0] = beyond[1];
        bin[2] = bin[3]; beyond[2] = beyond[3];
        if (k > 0) {
            wave_find_bin<true>(h, (uint32_t)k, lane, bin[0], beyond[0], in_bin);
            wave_find_bin<false>(h, (uint32_t)k, lane, bin[2], beyond[2], in_bin);
        }
        if (lane == 0) target[wave] = bin[0] | (bin[1] << 8) | (bin[2] << 16) | (bin[3] << 24);
    }
    __syncthreads();
    for (int i = tid; i < C * 4 * 256; i += CK_NT) cnt[i] = 0;
    uint32_t tg[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        tg[e] = target[lr * V + e];
        set_range(e, (tg[e] >> 8) & 255u, tg[e] >> 24);
    }
    __syncthreads();
    // sweep two: counts of the low byte inside each target bin (slot 1 and 3: the bins of the (k+1)-th;
    // slots 0 and 2 only where the k-th lies in another bin)
    ck_sweep<V, LPR>(col, D, T, 1, row0, [&](int e, uint32_t key) {
        const uint32_t b = key >> 8;
        if (b - first[e] >= span[e]) {
            uint32_t *low = cnt + (lr * V + e) * 4 * 256 + (key & 255u);
            const uint32_t t = tg[e];
            if (b == ((t >> 8) & 255u)) atomicAdd(low + 256, 1u);
            else if (b == (t & 255u)) atomicAdd(low, 1u);
            if (b == t >> 24) atomicAdd(low + 3 * 256, 1u);
            else if (b == ((t >> 16) & 255u)) atomicAdd(low + 2 * 256, 1u);
        }
    });
    __syncthreads();
    if (wave >= C) return;
    const uint32_t *low = cnt + wave * 4 * 256;
    uint32_t lb, bey, in_bin, key[4] = {0, 0, 0, 0};
    wave_find_bin<true>(low + 256, K1 - beyond[1], lane, lb, bey, in_bin);
    key[1] = (bin[1] << 8) | lb;
    wave_find_bin<false>(low + 3 * 256, K1 - beyond[3], lane, lb, bey, in_bin);
    key[3] = (bin[3] << 8) | lb;
    if (k > 0) {
        wave_find_bin<true>(low + (bin[0] == bin[1] ? 256 : 0), (uint32_t)k - beyond[0], lane, lb, bey, in_bin);
        key[0] = (bin[0] << 8) | lb;
        wave_find_bin<false>(low + (bin[2] == bin[3] ? 3 : 2) * 256, (uint32_t)k - beyond[2], lane, lb, bey, in_bin);
        key[2] = (bin[2] << 8) | lb;
    }
    if (lane == 0) ck_store(out, g * C + wave, k, key);
}

// consecutive groups on one XCD: block b of 8 n runs on XCD b mod 8
__device__ __forceinline__ int ck_spread(int b, int n) { return (n & 7) == 0 ? (b & 7) * (n >> 3) + (b >> 3) : b; }

template <int V, int LPR>
__global__ __launch_bounds__(CK_NT) __attribute__((amdgpu_waves_per_eu(LPR == 2 ? 4 : 8)))
void kvq_calib_channels(const uint16_t *__restrict__ k_cal, int T, int D, int k, int groups, const CkOut out)
{
    __shared__ CkLds<V, LPR> lds;
    ck_two_sweeps<V, LPR>(k_cal, T, D, k, ck_spread((int)blockIdx.x, groups), lds, out);
}

// ---- one sweep, with scratch memory -------------------------------------------------------------------------
// Whole lines: a workgroup reads 64 channels (128 bytes) of a part of the rows.  A sample bounds the order statistics so
// that one in thirty keys lies beyond the bounds; those are listed per channel and side in the scratch memory, and a second
// launch finds the order statistics among them.  Where many columns (below) meet at a bound, a crowd of equal keys, the keys strictly beyond
// the bounds are listed and those on them counted.  Lists that were too short for a part of the rows (rows of larger keys, all in one part) are
// made good by that launch from the part's rows.  Channels whose sample misled otherwise (too few keys beyond the bounds, or more than
// CL_ALL) take the two sweeps there.
// The bounds: every 16th row, a row of each sixteen picked by a hash, goes to one of 128 columns of threads, which keep
// their largest and smallest key per channel; the r-th largest of the 128 column maxima is a lower bound of the sample's
// r-th largest.  With r0 = (k + 1) / 16 of the order statistics' elements expected in the sample, r = r0 + 5 sqrt(r0) + 4 misses
// in about one call in a thousand.
// A lane lists a key in a column of LDS of its own (no atomic addition whose result it would wait for: that kept one sweep over
// 16 channels a workgroup no faster than two); full columns go to the channels' lists.
// Whole calls, us, two sweeps / one: 32768 x 4096 209 / 103 (of it 70 + 12 in the two launches; the sweep runs at 5.4 TB/s, what this
// access pattern reaches alone), 32768 x 1024 111 / 61, 32768 x 5120 359 / 128.  A third of the first launch is the start, the sample
// and the bounds.  Keys that a sample describes less well, 32768 x 4096, two sweeps / one: multiples of 1/2 367 / 137, constant channels 700 / 112, half of
// the keys zero 291 / 145, the last sixteenth of the rows fifty times as large 186 / 144, rows that grow sixfold 194 / 169, one channel of a layer whose
// sampled rows alone stand out 210 / 184 (all its channels: 205 / 364, which is the worst).  Outliers past the lists, from 1.3 % at 32768 rows
// on, take the two sweeps from the start (2 %: 224).
constexpr int CL_C = 64;                 // channels of a workgroup
constexpr int CL_LPR = 8;                // lanes of 8 channels to a row
constexpr int CL_COLS = CK_NT / CL_LPR;
constexpr int CL_CAP = 416;              // keys of a channel's side that a part lists
constexpr int CL_SLOTS = 12;             // keys that a lane holds
constexpr int CL_ALL = 1536;             // keys of a channel's side in all parts that the second launch takes
constexpr int CL_MAX_PARTS = 32;

constexpr uint32_t CL_NONE = 0xFFFFu;    // instead of a list's length: the bounds are of no use

struct CkPlan {
    int groups, parts, rows, rank;       // rows of a part; rank r of the bounds among the column maxima
};
// Of (64 channels, part), by [2 c + side]; on side 0 complements stand for the keys, so that either side is after the largest.
struct CkLists {
    uint16_t *keys;                      // [CL_CAP]
    uint32_t *counts;                    // keys beyond the bound, which the list holds up to CL_CAP, and << 16 those on it (0: they are listed)
    uint32_t *least;                     // the smallest key that is listed
};
constexpr int64_t CL_BYTES = CL_CAP * 2 + 2 * 4;

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 ck_two(uint32_t w) { return __builtin_bit_cast(u16x2, w); }
__device__ __forceinline__ uint32_t ck_word(u16x2 v) { return __builtin_bit_cast(uint32_t, v); }

// An x that at least `rank` of 128 keys reach, and hardly more than that where the keys allow it: built from the highest bit
// down, until at most an eighth of `rank` are too many (n: how many reach it).  Eight neighbouring lanes hold the keys, two to a word.
__device__ __forceinline__ uint32_t ck_bound(const u16x2 (&v)[8], uint32_t rank, uint32_t &n)
{
    const u16x2 one = ck_two(0x00010001u);
    uint32_t x = 0;
    n = 2 * 64;
#pragma unroll 1
    for (int bit = 15; bit >= 0 && __ballot(n > rank + (rank >> 3)) != 0ull; --bit) {
        const uint32_t y = x | (1u << bit);
        const u16x2 yy = ck_two(y | y << 16);
        u16x2 below = ck_two(0u);
#pragma unroll
        for (int u = 0; u < 8; ++u) below += __builtin_elementwise_min(__builtin_elementwise_sub_sat(yy, v[u]), one);
        uint32_t c = 16u - (below.x + below.y);
        c += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0xB1, 0xf, 0xf, false);       // lane ^ 1
        c += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0x4E, 0xf, 0xf, false);       // lane ^ 2
        c += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0x141, 0xf, 0xf, false);      // the other four of the eight
        if (c >= rank) { x = y; n = c; }
    }
    return x;
}

__global__ __launch_bounds__(CK_NT) void kvq_calib_list(const uint16_t *__restrict__ k_cal, int T, int D, const CkPlan plan,
                                                        const CkLists lists)
{
    __shared__ __attribute__((aligned(16))) uint16_t chan[2 * CL_C][CL_CAP];     // the channels' lists; first the column extremes
    __shared__ uint32_t mine[CL_SLOTS][CK_NT];
    __shared__ uint32_t n_listed[2 * CL_C], n_equal[2 * CL_C];
    __shared__ uint32_t top_s[CL_C], bot_s[CL_C];
    __shared__ int crowd_s;
    static_assert(sizeof(chan) >= 2 * CL_C * CL_COLS * 2, "the column extremes fit");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = ck_spread((int)blockIdx.x, plan.groups * plan.parts), g = b / plan.parts, part = b % plan.parts;
    const int lr = tid % CL_LPR, col = tid / CL_LPR;
    const uint16_t *base = k_cal + (int64_t)g * CL_C + lr * 8;
    const int t0 = part * plan.rows, t1 = t0 + plan.rows < T ? t0 + plan.rows : T;
    constexpr int U = 4;
    CkVec<8> v[U];
    auto load = [&](int i0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * CL_COLS;
            v[u] = ck_load<8>(base + (int64_t)(i < t1 ? i : t1 - 1) * D);
        }
    };
    // column extremes of the sample
    {
        const int n_sample = T / CK_STRIDE;
        u16x2 mx[4], mn[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) { mx[w] = ck_two(0u); mn[w] = ck_two(0xFFFFFFFFu); }
        for (int i0 = col; i0 < n_sample; i0 += 8 * CL_COLS) {
            CkVec<8> v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + u * CL_COLS < n_sample ? i0 + u * CL_COLS : i0;
                const int row = i * CK_STRIDE + (int)(((uint32_t)i * 2654435761u) >> 28);
                v[u] = ck_load<8>(base + (int64_t)row * D);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const u16x2 key = ck_two(ck_keys(v[u].w[w]));          // (a row taken twice changes no extreme)
                    mx[w] = __builtin_elementwise_max(mx[w], key);
                    mn[w] = __builtin_elementwise_min(mn[w], key);
                }
        }
        uint16_t *ext = &chan[0][0];                                      // [2 channel + side][column]
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint16_t *e = ext + (lr * 8 + 2 * w + h) * 2 * CL_COLS + col;
                e[0] = (uint16_t)~mn[w][h];                               // (smallest keys as largest complements)
                e[CL_COLS] = mx[w][h];
            }
    }
    if (tid < 2 * CL_C) n_listed[tid] = n_equal[tid] = 0;
    if (tid == 0) crowd_s = 0;
    load(t0 + col);
    __syncthreads();
    {
        static_assert(CK_NT / 8 == 2 * CL_C && CL_COLS == 128, "eight lanes per channel and side, sixteen columns each");
        const int i = tid >> 3;
        const uint4 *from = (const uint4 *)(&chan[0][0] + i * CL_COLS) + 2 * (tid & 7);
        const uint4 p = from[0], q = from[1];
        const u16x2 ext[8] = {ck_two(p.x), ck_two(p.y), ck_two(p.z), ck_two(p.w), ck_two(q.x), ck_two(q.y), ck_two(q.z), ck_two(q.w)};
        uint32_t n;
        const uint32_t x = ck_bound(ext, (uint32_t)plan.rank, n);
        if ((tid & 7) == 0) {
            if (i & 1) top_s[i >> 1] = x;
            else bot_s[i >> 1] = (~x) & 0xFFFFu;
            if (n > (uint32_t)plan.rank + ((uint32_t)plan.rank >> 3) + 4u) crowd_s = 1;         // (a few more keys do no harm)
        }
    }
    __syncthreads();
    if (tid < CL_C) {
        if (top_s[tid] <= bot_s[tid] + 1u) crowd_s = 1;
        if (top_s[tid] < bot_s[tid]) n_listed[2 * tid] = n_listed[2 * tid + 1] = CL_NONE;
    }
    __syncthreads();
    // keys between the bounds, with a crowd also those on them, are passed over: key - first <= less (all, where the bounds are of no use)
    const uint32_t crowd = (uint32_t)__builtin_amdgcn_readfirstlane(crowd_s);
    u16x2 first[4], less[4];
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t c = lr * 8 + 2 * w + h, tb = top_s[c], bb = bot_s[c];
            first[w][h] = (unsigned short)(tb < bb ? 0u : bb + 1u - crowd);
            less[w][h] = (unsigned short)(tb < bb ? 0xFFFFu : tb - bb - 2u + 2u * crowd);
        }
    uint32_t *slot = &mine[0][tid];
    auto flush = [&]() {
        const int n = (int)((slot - &mine[0][tid]) / CK_NT);
        for (int s = 0; __ballot(s < n) != 0ull; ++s) {
            if (s < n) {
                const uint32_t e = mine[s][tid], key = e & 0xFFFFu, c = lr * 8 + (e >> 16);
                const uint32_t l = 2 * c + (key >= top_s[c] + crowd ? 1u : 0u);
                const uint32_t at = atomicAdd(&n_listed[l], 1u);
                if (at < CL_CAP) chan[l][at] = (uint16_t)key;
            }
        }
        slot = &mine[0][tid];
    };
    u16x2 off[2][4];                       // by side: keys that are not on the bound
#pragma unroll
    for (int w = 0; w < 4; ++w) off[0][w] = off[1][w] = ck_two(0u);
    uint32_t rows = 0;                     // in both halves
    auto sweep = [&](auto counted) {
        for (int i0 = t0 + col; i0 - col < t1; i0 += U * CL_COLS) {        // (every lane of a wavefront makes as many rounds)
            if (i0 - col > t0) load(i0);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (i0 + u * CL_COLS < t1) {
                    rows += 0x00010001u;
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const uint32_t key = ck_keys(v[u].w[w]);
                        const u16x2 at = (u16x2)(ck_two(key) - first[w]);
                        const uint32_t out = ck_word(__builtin_elementwise_sub_sat(at, less[w]));
                        if constexpr (decltype(counted)::value) {
                            const u16x2 one = ck_two(0x00010001u);
                            off[0][w] += __builtin_elementwise_min(at, one);
                            off[1][w] += __builtin_elementwise_min((u16x2)(at ^ less[w]), one);
                        }
                        if (out & 0xFFFFu) {
                            *slot = (key & 0xFFFFu) | (uint32_t)(2 * w) << 16;
                            slot += CK_NT;
                        }
                        if (out > 0xFFFFu) {
                            *slot = __builtin_amdgcn_alignbit((uint32_t)(2 * w + 1), key, 16);
                            slot += CK_NT;
                        }
                    }
                }
                if (__ballot(slot > &mine[CL_SLOTS - 8][tid]) != 0ull) flush();
            }
        }
    };
    if (crowd) {
        sweep(std::true_type{});
#pragma unroll
        for (int side = 0; side < 2; ++side)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                uint32_t on = rows - ck_word(off[side][w]);                // (up to 256 in a lane)
                for (int o = CL_LPR; o < 64; o <<= 1) on += __shfl_xor(on, o);
                if (lane < CL_LPR) {
                    atomicAdd(&n_equal[2 * (lr * 8 + 2 * w) + side], on & 0xFFFFu);
                    atomicAdd(&n_equal[2 * (lr * 8 + 2 * w + 1) + side], on >> 16);
                }
            }
    } else {
        sweep(std::false_type{});
    }
    flush();
    __syncthreads();
    const int64_t l0 = (int64_t)(g * plan.parts + part) * (2 * CL_C);
    if (tid < 2 * CL_C) {
        lists.counts[l0 + tid] = n_listed[tid] | n_equal[tid] << 16;
        lists.least[l0 + tid] = ((tid & 1) ? top_s[tid >> 1] : 0xFFFFu - bot_s[tid >> 1]) + crowd;
    }
    uint32_t *keys = (uint32_t *)(lists.keys + l0 * CL_CAP);
    for (int l = wave; l < 2 * CL_C; l += CK_NT / 64) {
        const int n = (int)(n_listed[l] < CL_CAP ? n_listed[l] : CL_CAP);
        for (int i = lane; 2 * i < n; i += 64) keys[l * (CL_CAP / 2) + i] = ((const uint32_t *)chan[l])[i];
    }
}

// The rank-th largest (x) of a wavefront's n keys in LDS (larger: further out), and how many are larger than it.  Two
// histograms of the keys between their smallest and their largest; hist: 256 words of the wavefront's.
__device__ __forceinline__ uint32_t ck_pick(const uint16_t *keys, uint32_t n, uint32_t rank, uint32_t *hist, int lane, uint32_t &larger)
{
    uint32_t lo = 0xFFFFu, hi = 0;
    for (uint32_t i = lane; i < n; i += 64) {
        const uint32_t v = keys[i];
        lo = v < lo ? v : lo;
        hi = v > hi ? v : hi;
    }
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t a = __shfl_xor(lo, o), b = __shfl_xor(hi, o);
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
    }
    const int bits = 32 - __builtin_clz((hi - lo) | 1u), sh = bits > 8 ? bits - 8 : 0;
    auto count = [&](auto f) {
        *(uint4 *)(hist + 4 * lane) = uint4{0, 0, 0, 0};
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (uint32_t i = lane; i < n; i += 64) f((uint32_t)keys[i] - lo);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    auto add = [&](uint32_t bin) { __hip_atomic_fetch_add(&hist[bin], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT); };
    uint32_t bin, in_bin, low = 0, beyond = 0;
    count([&](uint32_t d) { add(d >> sh); });
    wave_find_bin<true>(hist, rank, lane, bin, larger, in_bin);
    if (sh > 0) {
        count([&](uint32_t d) {
            if (d >> sh == bin) add(d & ((1u << sh) - 1u));
        });
        wave_find_bin<true>(hist, rank - larger, lane, low, beyond, in_bin);
        larger += beyond;
    }
    return lo + (bin << sh) + low;
}

// A wavefront per channel and side, eight channels a workgroup: the order statistics among the listed keys.
struct CkPickLds {
    __attribute__((aligned(16))) uint16_t keys[CK_NT / 64][CL_ALL];
    __attribute__((aligned(16))) uint32_t hist[CK_NT / 64][256];
};
__global__ __launch_bounds__(CK_NT) __attribute__((amdgpu_waves_per_eu(8)))
void kvq_calib_pick(const uint16_t *__restrict__ k_cal, int T, int D, int k, const CkPlan plan, const CkLists lists, const CkOut out)
{
    union Lds {
        CkPickLds pick;
        CkLds<8, 1> two;
    };
    __shared__ Lds lds;
    __shared__ uint32_t found[8][4];       // see ck_store
    __shared__ uint32_t again_s;           // parts whose keys did not fit into a list of this workgroup's
    __shared__ uint32_t least_s[CK_NT / 64], next_s[CK_NT / 64];
    __shared__ int failed;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g8 = ck_spread((int)blockIdx.x, (int)gridDim.x), side = wave & 1, c = g8 * 8 + (wave >> 1);
    const uint32_t K1 = (uint32_t)k + 1u;
    // this wavefront's list, by part in the lanes: keys of the part, up to it, on the bound
    const int64_t l0 = (int64_t)(c / CL_C) * plan.parts * (2 * CL_C) + 2 * (c % CL_C) + side;
    const uint32_t count = lane < plan.parts ? lists.counts[l0 + (int64_t)lane * (2 * CL_C)] : 0u, n = count & 0xFFFFu;
    const uint32_t least = lists.least[l0], over = (uint32_t)__ballot(n > CL_CAP);
    if (tid == 0) { failed = 0; again_s = 0; }
    __syncthreads();
    uint32_t sum = n, on = count >> 16;
    for (int o = 1; o < CL_MAX_PARTS; o <<= 1) {
        const uint32_t t = __shfl_up(sum, o);
        if (lane >= o) sum += t;
        on += __shfl_xor(on, o);
    }
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)sum, plan.parts - 1);
    on = (uint32_t)__builtin_amdgcn_readfirstlane((int)on);
    uint16_t *all = lds.pick.keys[wave];
    if (__ballot(n == CL_NONE) != 0ull || total + on < K1 || total > CL_ALL) {
        if (lane == 0) failed = 1;
    } else {
        if (lane == 0 && over != 0u) atomicOr(&again_s, over);
        constexpr int W = (CL_CAP / 2 + 63) / 64;      // words a lane reads of a list
        for (int p0 = 0; p0 < plan.parts; p0 += 4) {
            uint32_t e[4][W], n4[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int p = p0 + q < plan.parts ? p0 + q : p0;
                const uint32_t np = p0 + q < plan.parts ? (uint32_t)__builtin_amdgcn_readlane((int)n, p) : 0u;
                n4[q] = np <= CL_CAP ? np : 0u;
                const uint32_t *from = (const uint32_t *)(lists.keys + (l0 + (int64_t)p * (2 * CL_C)) * CL_CAP);
#pragma unroll
                for (int u = 0; u < W; ++u) e[q][u] = 2 * (64 * u + lane) < (int)n4[q] ? from[64 * u + lane] : 0u;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int p = p0 + q < plan.parts ? p0 + q : p0;
                uint16_t *to = all + (uint32_t)__builtin_amdgcn_readlane((int)sum, p) - (uint32_t)__builtin_amdgcn_readlane((int)n, p);
#pragma unroll
                for (int u = 0; u < W; ++u) {
                    const uint32_t i = 2 * (64 * u + lane), v = side ? e[q][u] : ~e[q][u];
                    if (i < n4[q]) to[i] = (uint16_t)v;
                    if (i + 1 < n4[q]) to[i + 1] = (uint16_t)(v >> 16);
                }
            }
        }
    }
    __syncthreads();
    if (failed) {
        ck_two_sweeps<8, 1>(k_cal, T, D, k, g8, lds.two, out);       // all eight channels
        return;
    }
    for (uint32_t left = again_s; left != 0u; left &= left - 1u) {
        const int p = __ffs((int)left) - 1, r1 = (p + 1) * plan.rows < T ? (p + 1) * plan.rows : T;
        const uint32_t at0 = (uint32_t)__builtin_amdgcn_readlane((int)sum, p) - (uint32_t)__builtin_amdgcn_readlane((int)n, p);
        if (lane == 0) {
            least_s[wave] = (over >> p) & 1u ? least : 0x20000u;       // (no key is that large)
            next_s[wave] = at0;
        }
        __syncthreads();
        for (int i = p * plan.rows + tid; i < r1; i += CK_NT) {
            const CkVec<8> v = ck_load<8>(k_cal + (int64_t)i * D + g8 * 8);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t key = (ck_keys(v.w[e >> 1]) >> (16 * (e & 1))) & 0xFFFFu;
#pragma unroll
                for (int sd = 0; sd < 2; ++sd) {
                    const uint32_t x = sd ? key : 0xFFFFu - key;
                    if (x >= least_s[2 * e + sd]) {
                        const uint32_t at = atomicAdd(&next_s[2 * e + sd], 1u);
                        if (at < CL_ALL) lds.pick.keys[2 * e + sd][at] = (uint16_t)x;
                    }
                }
            }
        }
        __syncthreads();
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // x: the (k+1)-th; xk: the k-th, the next key up where just k are larger, and otherwise the same
    uint32_t larger = total, x = least - 1u;                   // (too few beyond the bound: the bound)
    if (total >= K1) x = ck_pick(all, total, K1, lds.pick.hist[wave], lane, larger);
    uint32_t xk = x;
    if (larger == (uint32_t)k) {
        xk = 0xFFFFu;
        for (uint32_t i = lane; i < total; i += 64) {
            const uint32_t v = all[i];
            xk = v > x && v < xk ? v : xk;
        }
        for (int o = 32; o > 0; o >>= 1) {
            const uint32_t a = __shfl_xor(xk, o);
            xk = a < xk ? a : xk;
        }
    }
    if (lane == 0) {
        found[wave >> 1][side ? 1 : 3] = side ? x : (~x & 0xFFFFu);
        found[wave >> 1][side ? 0 : 2] = side ? xk : (~xk & 0xFFFFu);
    }
    __syncthreads();
    if (lane == 0 && side == 0) {
        const uint32_t key[4] = {found[wave >> 1][0], found[wave >> 1][1], found[wave >> 1][2], found[wave >> 1][3]};
        ck_store(out, c, k, key);
    }
}

// Outliers per side and channel; false: not a call.
bool ck_count(int T, int D, float fraction, int &k)
{
    if (T < 1 || D < 1 || !(fraction >= 0.0f) || !(fraction < 1.0f)) return false;
    k = (int)floorf(fraction * 0.5f * (float)T + 0.5f);
    return 2 * (int64_t)k < T;
}

// Whether and how a call takes the one sweep.
bool ck_plan(const void *k_cal, int T, int D, int k, CkPlan &plan)
{
    if (D % CL_C != 0 || ((uintptr_t)k_cal & 15)) return false;
    // The sample, the bounds and the second launch cost 25 us, which short calls would not get back.  Whole calls, us, two sweeps / one,
    // without outliers and with 1 %: 24576 x 128 60.5 / 57.6, 62.1 / 59.3, 20000 x 128 53.4 / 57.2, 55.3 / 58.4; 16384 x 256 57.0 / 55.3,
    // 58.8 / 56.8; 16384 x 1024 59.1 / 51.9, 63.5 / 53.9; 12000 x 512 48.8 / 56.1, 50.6 / 56.8; 8192 x 2048 46.1 / 50.0, 52.2 / 51.3, 9000 x 2048
    // 51.4 / 49.4, 54.5 / 50.9; 8192 x 4096 56.5 / 55.9, 67.5 / 58.6; 4096 x 5120 56.2 / 57.7, 70.8 / 60.3, 0.1 % 53.7 / 58.4, 0.5 % 58.0 / 59.0;
    // 4096 x 4096 41.5 / 51.1, 48.5 / 52.9.
    const int64_t all_keys = (int64_t)T * D;
    if (!(T >= 24576 || (T >= 16384 && D >= 256) || (T >= 8192 && all_keys > (16 << 20)) ||
          (k >= 16 && T >= 4096 && all_keys >= (20 << 20))))
        return false;
    const int n_sample = T / CK_STRIDE;
    const double r0 = (double)(k + 1) * n_sample / T, r = r0 + 5.0 * sqrt(r0) + 4.0;
    if (r > CL_COLS / 2) return false;
    plan.rank = (int)ceil(r);
    plan.groups = D / CL_C;
    // the share of keys beyond a bound, and how many that may be in a part and in all (1.7: the bound's own scatter)
    const double q = 1.0 - pow(1.0 - (double)plan.rank / CL_COLS, (double)CL_COLS / n_sample);
    const double all = 1.7 * q * T;
    if (all + 4.5 * sqrt(all) > CL_ALL) return false;
    // a workgroup per compute unit, or twice as many where the lists would not hold so long a part's keys
    for (int rounds = 1; rounds <= 2; ++rounds) {
        plan.parts = rounds * kvq_cu_count() / plan.groups;
        if (plan.parts > CL_MAX_PARTS) plan.parts = CL_MAX_PARTS;
        if (plan.parts < 1) plan.parts = 1;
        plan.rows = (T + plan.parts - 1) / plan.parts;
        plan.parts = (T + plan.rows - 1) / plan.rows;
        const double part = 1.7 * q * plan.rows;
        if (part + 4.5 * sqrt(part) + 8 <= CL_CAP) return true;
    }
    return false;
}

}  // namespace

extern "C" int64_t kvq_calibrate_key_channels_workspace_bytes(int32_t T, int32_t D, float outlier_fraction)
{
    CkPlan plan;
    int k;
    if (T > 32768 || !ck_count(T, D, outlier_fraction, k) || !ck_plan(nullptr, T, D, k, plan)) return 0;
    return (int64_t)plan.groups * plan.parts * (2 * CL_C) * CL_BYTES;
}

extern "C" kvq_status kvq_calibrate_key_channels_ws(const uint16_t *d_k_cal, int32_t T, int32_t D, float outlier_fraction,
                                                    uint16_t *d_s, uint16_t *d_z, uint16_t *d_lo, uint16_t *d_hi,
                                                    void *d_workspace, int64_t workspace_bytes, void *stream)
{
    if (!d_k_cal || !d_s || !d_z || !d_lo || !d_hi || ((uintptr_t)d_k_cal & 1)) return KVQ_ERR_INVALID_ARG;
    if (T < 1 || D < 1 || !(outlier_fraction >= 0.0f) || !(outlier_fraction < 1.0f)) return KVQ_ERR_INVALID_ARG;
    if (T > 32768) return KVQ_ERR_UNSUPPORTED;
    int k;
    if (!ck_count(T, D, outlier_fraction, k)) return KVQ_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    const CkOut out{d_s, d_z, d_lo, d_hi};
    CkPlan plan;
    if (d_workspace && ((uintptr_t)d_workspace & 15) == 0 && ck_plan(d_k_cal, T, D, k, plan) &&
        workspace_bytes >= kvq_calibrate_key_channels_workspace_bytes(T, D, outlier_fraction)) {
        const int64_t n = (int64_t)plan.groups * plan.parts, n_lists = n * (2 * CL_C);
        uint16_t *keys = (uint16_t *)d_workspace;
        uint32_t *counts = (uint32_t *)(keys + n_lists * CL_CAP);
        const CkLists lists{keys, counts, counts + n_lists};
        kvq_calib_list<<<(unsigned)n, CK_NT, 0, s>>>(d_k_cal, T, D, plan, lists);
        kvq_calib_pick<<<(unsigned)(D / 8), CK_NT, 0, s>>>(d_k_cal, T, D, k, plan, lists, out);
        KVQ_HIP_CHECK(hipGetLastError());
        return KVQ_OK;
    }
    // The widest group that divides D, whose loads are aligned, and that still gives a workgroup per compute
    // unit (a group is swept by one workgroup from end to end).  Measured on 32768 x 4096: groups of 32
    // channels (64-byte pieces, half the compute units) 272 us, of 16 182 us, of 8 (16-byte pieces) 248 us.
    const int64_t cus = kvq_cu_count();
    auto fits = [&](int v, int c) {
        return D % c == 0 && ((uintptr_t)d_k_cal & (2 * v - 1)) == 0 && (c == 1 || (int64_t)D / c >= cus);
    };
#define LAUNCH_CK(V, LPR)                                                                                          \
    kvq_calib_channels<V, LPR><<<D / ((V) * (LPR)), CK_NT, 0, s>>>(d_k_cal, T, D, k, D / ((V) * (LPR)), out)
    if (fits(8, 16)) LAUNCH_CK(8, 2);
    else if (fits(8, 8)) LAUNCH_CK(8, 1);
    else if (fits(4, 4)) LAUNCH_CK(4, 1);
    else if (fits(2, 2)) LAUNCH_CK(2, 1);
    else LAUNCH_CK(1, 1);
#undef LAUNCH_CK
    KVQ_HIP_CHECK(hipGetLastError());
    return KVQ_OK;
}

extern "C" kvq_status kvq_calibrate_key_channels(const uint16_t *d_k_cal, int32_t T, int32_t D, float outlier_fraction,
                                                 uint16_t *d_s, uint16_t *d_z, uint16_t *d_lo, uint16_t *d_hi,
                                                 void *stream)
{
    return kvq_calibrate_key_channels_ws(d_k_cal, T, D, outlier_fraction, d_s, d_z, d_lo, d_hi, nullptr, 0, stream);
}
