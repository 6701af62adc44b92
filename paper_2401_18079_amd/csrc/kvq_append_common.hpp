// What the append kernels share.
#pragma once
#include "kvq_select.hpp"
#include "kvq_append_keys.hpp"

namespace {

// Code of a normalised value: the number of thresholds it has reached (a compare and an add with carry each),
// or, beyond the range in which that is the nearest signpost, the exhaustive search (KVQ_CODE_RANGE).  The
// search costs four instructions per signpost; a token's channels are within the range all but always.
template <int NE>
struct KvqCoder {
    float thr[NE - 1], range;
    const float *lut;
    __device__ __forceinline__ KvqCoder(const float *thresholds, const float *signposts) : lut(signposts)
    {
#pragma unroll
        for (int j = 0; j < NE - 1; ++j) thr[j] = thresholds[j];
        range = (thr[0] == thr[0]) ? KVQ_CODE_RANGE : -1.0f;
    }
    __device__ __forceinline__ bool far(float xn) const { return !(__builtin_fabsf(xn) <= range); }
    __device__ __forceinline__ int count(float xn) const            // not far(xn) only
    {
        int code = 0;
#pragma unroll
        for (int j = 0; j < NE - 1; ++j) code += (xn >= thr[j]) ? 1 : 0;
        return code;
    }
    __device__ __forceinline__ int search(float xn) const
    {
        float sp;
        return kvq_nearest<NE>(lut, xn, sp);
    }
    __device__ __forceinline__ int operator()(float xn) const
    {
        if (NE == 4) return search(xn);       // (as short; with the branch below 5 % slower in the routines for any width)
        int code = count(xn);
        const bool f = far(xn);
        if (__ballot(f) != 0ull) {
            if (f) code = search(xn);
        }
        return code;
    }
};

// Number of Key outliers of each new token (threshold test only).  One wavefront per token, eight
// channels per lane and pass (16-byte loads of the fp16 vector, D is a multiple of 128): no barriers.  Bound by its loads' latency in small calls
// (64 tokens of 4096 channels, Keys and Values 16.8 us with fp32 thresholds, 64 bytes of them per 16 of Keys / 15.4), by vector issue beside the Value
// kernel in large ones (4096 tokens 49.4 / 48.5).
// PACKED: for kvq_k_bulk, which reads the channels' first and last keys too.  The other Key kernels read the fp32 thresholds, which this one then
// finds for them: two tokens, 4 bits, us per Key append, packed / fp32 thresholds: 16 heads 8.2 / 8.0, 32 heads 10.2 / 9.9, 64 heads 14.6 / 13.9.
constexpr int KVQ_COUNT_NT = 256;
template <bool PACKED>
__device__ __forceinline__ void k_count_token(const void *params, int D, const uint16_t *k_new, uint32_t *cnt, const int t)
{
    KvqParamsView pv = kvq_params_view(params, D);
    const int lane = threadIdx.x & 63;
    uint32_t mine = 0;
    auto one = [&](int c) {
        const float x = kvq_h2f(k_new[(int64_t)t * D + c]);
        return ((x < pv.lo[c]) | (x > pv.hi[c])) ? 1u : 0u;
    };
    const uint4 *row = (const uint4 *)(k_new + (int64_t)t * D);
    if ((uintptr_t)k_new & 15) {          // input not 16-byte aligned: one channel per lane and pass
        for (int c = lane; c < D; c += 64) mine += one(c);
    } else if constexpr (!PACKED) {
        const float4 *lo4 = (const float4 *)pv.lo, *hi4 = (const float4 *)pv.hi;
        for (int v = lane; v < D / 8; v += 64) {
            const uint4 h = row[v];
            const float4 la = lo4[2 * v], lb = lo4[2 * v + 1], ha = hi4[2 * v], hb = hi4[2 * v + 1];
            const uint32_t w[4] = {h.x, h.y, h.z, h.w};
            const float lo[8] = {la.x, la.y, la.z, la.w, lb.x, lb.y, lb.z, lb.w};
            const float hi[8] = {ha.x, ha.y, ha.z, ha.w, hb.x, hb.y, hb.z, hb.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float x = kvq_h2f((uint16_t)(w[e >> 1] >> (16 * (e & 1))));
                mine += ((x < lo[e]) | (x > hi[e])) ? 1u : 0u;
            }
        }
    } else {
        // packed keys against the channels' first and last that are no outlier (KvqKeyParams); one by one where the range ends at the code range
        // and something lies beyond.  NaN lies beyond every range and is no outlier.
        const KvqKeyParams kp = kvq_key_params(params, D);
        const uint4 *first = (const uint4 *)kp.first, *last = (const uint4 *)kp.last;
        for (int v = lane; v < D / 8; v += 64) {
            const uint4 h = row[v], f = first[v], l = last[v];
            uint32_t narrow = kp.narrow[v];
            asm("" : "+v"(narrow));      // (requested with the others, not where it is needed)
            const uint32_t w[4] = {h.x, h.y, h.z, h.w}, fw[4] = {f.x, f.y, f.z, f.w}, lw[4] = {l.x, l.y, l.z, l.w};
            s16x2 out = {0, 0};           // less the outliers among the even and the odd channels
            half2_t odd = {(half_t)0, (half_t)0};                          // NaN: one of the elements is
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const s16x2 s = vp_keys(w[i]);
                out += vp_pair(vp_less(s, vp_pair(fw[i])) | vp_less(vp_pair(lw[i]), s));
                odd = __builtin_elementwise_maximum(odd, __builtin_bit_cast(half2_t, w[i]));
            }
            int n = -(out.x + out.y);
            if (n != 0 && narrow != 0) {
                n = 0;
                for (int e = 0; e < 8; ++e) n += one(8 * v + e);
            } else if (!(odd.x == odd.x) || !(odd.y == odd.y)) {
                s16x2 nan = {0, 0};       // less their number
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const s16x2 s = vp_keys(w[i]);
                    nan += vp_pair(vp_less(vp_both(31744), s) | vp_less(s, vp_both(-31745)));
                }
                n += nan.x + nan.y;
            }
            mine += (uint32_t)n;
        }
    }
    for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o);
    if (lane == 0) cnt[t] = mine;
}
// In bulk a Value kernel's first `wgs` workgroups count the Key outliers of the same tokens (a wavefront per token):
// reading the Keys and the thresholds, latency that the Values' arithmetic covers.  wgs = 0: Values only.
struct KeyCount {
    int wgs;
    const uint16_t *k_new;
    uint32_t *cnt;
};

constexpr int KVQ_V_CAND = 128;              // candidates per side that a wavefront looks through (two per lane)
constexpr uint32_t KVQ_V_BOUNDED = 52;       // outliers per side up to which the thresholds are bounded first

}  // namespace

// Workgroup b of a launch runs on XCD b mod 8.  The codes of 64 consecutive tokens (or pairs) share lines, 16 bytes each: a launch of
// kvq_xcd_grid(n) workgroups takes its n pieces of work in this order, so that an XCD has neighbours and its L2 puts their bytes together.
// (The last ones may have none: place >= n.)
__host__ __device__ inline unsigned kvq_xcd_grid(unsigned n) { return (n + 7) & ~7u; }
__device__ __forceinline__ unsigned kvq_xcd_place(unsigned b, unsigned grid) { return (b & 7) * (grid >> 3) + (b >> 3); }

// Widest bulk appends of kvq_v_pair.hip and kvq_k_bulk.hip: one wavefront per 1024 channels.
constexpr int KVQ_BULK_MAX_WAVES = 8;
// Launches the pair kernel over `pairs` pairs of tokens (and the counting workgroups).  D a multiple of 1024, up to 1024 KVQ_BULK_MAX_WAVES;
// k_side_v at most KVQ_V_BOUNDED; d_v_new 16-byte aligned.
__attribute__((visibility("hidden"))) void kvq_v_pair_launch(const kvq_cache *cache, const uint16_t *d_v_new, int T, unsigned pairs,
                                                             int count_wgs, const uint16_t *k_new, uint32_t *k_count, hipStream_t s);
// Launches kvq_k_bulk; `counts`: the tokens' outlier counts, in a workspace with room for a multiple of four.  D a multiple of 1024 up to
// 1024 KVQ_BULK_MAX_WAVES; d_k_new 16-byte aligned.
__attribute__((visibility("hidden"))) void kvq_k_bulk_launch(const kvq_cache *cache, const uint16_t *d_k_new, int T, const uint32_t *counts,
                                                             hipStream_t s);
// Tokens of a workgroup's run.
inline int kvq_k_bulk_run(int bits, int D, int T)
{
    // workgroups that the compute units hold at once (188 registers with 4 bits, 128 or fewer with 2 and 3)
    const int waves = D / 1024, per_cu = (bits == 4 ? 8 : 16) / waves, most = kvq_cu_count() * (per_cu > 0 ? per_cu : 1);
    return (T + most - 1) / most;
}
