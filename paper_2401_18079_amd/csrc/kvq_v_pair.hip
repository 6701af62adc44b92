// Bulk Value append, a workgroup per pair of tokens (the two that share the dwords of their codes).
#include <type_traits>
#include "kvq_append_common.hpp"
#include "kvq_append_keys.hpp"

namespace {

// A lane has sixteen neighbouring channels of both tokens, so that the workgroup has one thread per sixteen channels (D a multiple of
// 1024), the fields of a lane are a run of whole dwords of the storage format and no code goes through LDS.  Elements stay in
// registers as 16-bit keys, two to a register, and everything that is done to each of them is done to two at once
// with packed 16-bit instructions:
//  * keys: x as a signed number in the order of the values (-0 directly below 0);
//  * the outlier thresholds as in v_quant_token4 - the k-th largest of 64 columns' maxima bounds the k-th largest key, the few
//    keys beyond are collected and the thresholds found among them with ballots -, but each of the four searches (two
//    tokens, two sides) by one wavefront for all;
//  * codes: the normalised value grows with x, so that the code of x is the number of keys K_j <= x where K_j is the smallest
//    fp16 number whose normalised value (the same fp32 steps) reaches the j-th threshold.  One lane per threshold and token
//    finds its K_j, next to where the inverse of the normalisation points; an element's code is a binary search of
//    log2 comparisons, each a saturating subtraction whose sign selects the next K_j.
// Tokens with crowds of equal keys (more candidates than the lists hold, thresholds that coincide) and thresholds at zero, which
// has two keys, take general_selection; far outliers are encoded one by one.  Same arithmetic, same
// results, as v_quant_token.
// us per Value append, the kernel with a token on four wavefronts and a lane per element (v_quant_token4) / this one, 1 % outliers:
// 4096 tokens of 4096 channels, 2 bits 46.8 / 23.9, 3 bits 51.5 / 26.5, 4 bits 56.5 / 29.6; of 5120, 4 bits 77.1 / 44.2; of 8192 116 / 55; 777 of
// 5120 22.5 / 15.0; 64 of 4096 13.8 / 11.3; 4096 of 3072 (the routine for any width before) 82.4 / 25.8.  Bound by vector issue, with six wavefronts
// a SIMD (five: 5120 channels 44.9 / 41.8 at first, 3 bits; eight, which spill: 40.9, but 4096 channels 30.3 against 29.2).

// Packed maxima over the wavefront (two numbers at once), in every lane.
__device__ __forceinline__ s16x2 vp_wave_max(s16x2 v)
{
    v = __builtin_elementwise_max(v, vp_pair(vp_dpp<0x128>(0u, vp_word(v))));
    v = __builtin_elementwise_max(v, vp_pair(vp_dpp<0x124>(0u, vp_word(v))));
    v = __builtin_elementwise_max(v, vp_pair(vp_dpp<0x122>(0u, vp_word(v))));
    v = __builtin_elementwise_max(v, vp_pair(vp_dpp<0x121>(0u, vp_word(v))));
    const int b = (int)vp_word(v);
    const s16x2 r0 = vp_pair((uint32_t)__builtin_amdgcn_readlane(b, 0)), r1 = vp_pair((uint32_t)__builtin_amdgcn_readlane(b, 16));
    const s16x2 r2 = vp_pair((uint32_t)__builtin_amdgcn_readlane(b, 32)), r3 = vp_pair((uint32_t)__builtin_amdgcn_readlane(b, 48));
    return __builtin_elementwise_max(__builtin_elementwise_max(r0, r1), __builtin_elementwise_max(r2, r3));
}

// Searches of a workgroup are numbered 2 token + side; side 1 works on complemented keys, so that either looks for the k-th largest.
struct VpLds {
    int col_max[4][64];                        // the largest keys of the 64 columns (lane l of every wavefront)
    uint32_t n_cand[4];
    uint16_t cand[4][KVQ_V_CAND];              // candidates, + 32768
    int bound[4];
    struct { int tau; uint32_t need, n_eq; } found[4];     // threshold; how many of its equals are taken, how many there are
    __attribute__((aligned(16))) uint32_t wave_red[3][KVQ_BULK_MAX_WAVES];       // of a wavefront's inliers (tokens packed): largest, complement of smallest; outliers
    uint32_t counts[17][2];                    // general_selection's rounds
    uint32_t eq[KVQ_BULK_MAX_WAVES][2];
    float lut[16];
};

// The outliers of both tokens where the lists do not serve: thresholds by bisection over all keys (-0 as 0), a barrier a bit; of a
// threshold's equals the first in channel order.  Returns the outliers: bit w + 8 token + 16 half is half `half` of this lane's
// word w.
__device__ __forceinline__ uint32_t general_selection(VpLds &lds, const s16x2 (&s)[2][8], uint32_t K)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, NT = blockDim.x;
    const u16x2v one = {1, 1};
    u16x2v key[2][8];
#pragma unroll
    for (int tok = 0; tok < 2; ++tok)
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const u16x2v not_neg_zero = __builtin_elementwise_min(__builtin_bit_cast(u16x2v, ~vp_word(s[tok][w])), one);
            const uint32_t canonical = vp_word(s[tok][w] + (short)1 - __builtin_bit_cast(s16x2, not_neg_zero));
            key[tok][w] = __builtin_bit_cast(u16x2v, canonical ^ 0x80008000u);
        }
    for (int i = tid; i < 17 * 2; i += NT) (&lds.counts[0][0])[i] = 0;
    __syncthreads();
    uint32_t x[4] = {0, 0, 0, 0}, gt[4] = {0, 0, 0, 0};
    for (int bit = 15; bit >= -1; --bit) {               // (the last round: how many exceed the thresholds themselves)
#pragma unroll
        for (int tok = 0; tok < 2; ++tok) {
            const unsigned short yt = (unsigned short)(bit >= 0 ? (x[2 * tok] | (1u << bit)) - 1u : x[2 * tok]);
            const unsigned short yb = (unsigned short)(bit >= 0 ? (x[2 * tok + 1] | (1u << bit)) - 1u : x[2 * tok + 1]);
            const u16x2v xt = {yt, yt}, xb = {yb, yb};
            u16x2v a = {0, 0}, b = {0, 0};
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                a += __builtin_elementwise_min(__builtin_elementwise_sub_sat(key[tok][w], xt), one);
                b += __builtin_elementwise_min(__builtin_elementwise_sub_sat((u16x2v)(~key[tok][w]), xb), one);
            }
            // keys above either threshold, the token's sides packed
            const uint32_t sum = (uint32_t)__builtin_amdgcn_readlane((int)vp_scan((uint32_t)(a.x + a.y) | (uint32_t)(b.x + b.y) << 16), 63);
            if (lane == 0) atomicAdd(&lds.counts[15 - bit][tok], sum);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t n = (lds.counts[15 - bit][i >> 1] >> (16 * (i & 1))) & 0xFFFFu;
            if (bit < 0) gt[i] = n;
            else if (n >= K) x[i] |= 1u << bit;
        }
    }
    // equals before this lane's channels
    uint32_t before[2];
#pragma unroll
    for (int tok = 0; tok < 2; ++tok) {
        uint32_t mine = 0;
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const u16x2v k = key[tok][w];
            mine += (k.x == x[2 * tok] ? 1u : 0u) + (k.y == x[2 * tok] ? 1u : 0u);
            mine += ((0xFFFFu ^ k.x) == x[2 * tok + 1] ? 0x10000u : 0u) + ((0xFFFFu ^ k.y) == x[2 * tok + 1] ? 0x10000u : 0u);
        }
        const uint32_t upto = vp_scan(mine);
        before[tok] = upto - mine;
        if (lane == 63) lds.eq[wave][tok] = upto;
    }
    __syncthreads();
    uint32_t out = 0;
#pragma unroll
    for (int tok = 0; tok < 2; ++tok) {
        for (int w = 0; w < wave; ++w) before[tok] += lds.eq[w][tok];
        const uint32_t tt = x[2 * tok], tb = x[2 * tok + 1], need_t = K - gt[2 * tok], need_b = K - gt[2 * tok + 1];
        const bool same = tt == 0xFFFFu - tb;
        uint32_t rt = before[tok] & 0xFFFFu, rb = before[tok] >> 16;
#pragma unroll
        for (int w = 0; w < 8; ++w) {
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const uint32_t k = half ? key[tok][w].y : key[tok][w].x, inv = 0xFFFFu ^ k;
                const bool eq_t = k == tt, eq_b = inv == tb;
                const bool is_top = k > tt || (eq_t && rt < need_t);
                // thresholds coincide: the lower outliers take the equal keys that follow the upper ones'
                const bool is_bot = inv > tb || (eq_b && (same ? (rb >= need_t && rb < need_t + need_b) : rb < need_b));
                rt += eq_t ? 1u : 0u;
                rb += eq_b ? 1u : 0u;
                out |= (is_top || is_bot) ? 1u << (w + 8 * tok + 16 * half) : 0u;
            }
        }
    }
    return out;
}

// Of the keys that equal a threshold only the first need[i] in channel order are outliers: takes the others out of `outl`.
__device__ __forceinline__ uint32_t drop_equals(VpLds &lds, const s16x2 (&s)[2][8], uint32_t outl)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t eq[2] = {0, 0}, before[2];                  // by side; bits as in the result
#pragma unroll
    for (int tok = 0; tok < 2; ++tok) {
        const s16x2 tt = vp_both(lds.found[2 * tok].tau), tb = vp_both(~lds.found[2 * tok + 1].tau);
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            // (outliers on or beyond a threshold: equal where not beyond)
            eq[0] |= ~(vp_less(s[tok][w], tt) | vp_less(tt, s[tok][w])) & (0x00010001u << (w + 8 * tok));
            eq[1] |= ~(vp_less(s[tok][w], tb) | vp_less(tb, s[tok][w])) & (0x00010001u << (w + 8 * tok));
        }
    }
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const uint32_t mine = (uint32_t)__popc(eq[side] & 0x00FF00FFu) | (uint32_t)__popc(eq[side] & 0xFF00FF00u) << 16;
        const uint32_t upto = vp_scan(mine);
        before[side] = upto - mine;
        if (lane == 63) lds.eq[wave][side] = upto;
    }
    __syncthreads();
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        for (int w = 0; w < wave; ++w) before[side] += lds.eq[w][side];
#pragma unroll
        for (int tok = 0; tok < 2; ++tok) {
            const uint32_t need = lds.found[2 * tok + side].need;
            uint32_t rank = (before[side] >> (16 * tok)) & 0xFFFFu, left = (eq[side] >> (8 * tok)) & 0x00FF00FFu;
            while (left != 0u) {                         // in channel order: words, then halves
                const int w = __ffs((int)((left | left >> 16) & 0xFFu)) - 1;
                const uint32_t bit = 1u << w & left ? 1u << w : 0x10000u << w;
                left &= ~bit;
                if (rank++ >= need) outl &= ~(bit << (8 * tok));
            }
        }
    }
    return outl;
}

template <int BITS, class SP>
__global__ __launch_bounds__(64 * KVQ_BULK_MAX_WAVES) __attribute__((amdgpu_waves_per_eu(6))) void kvq_v_pair(const void *__restrict__ params, int D, int64_t cap, int64_t n0,
                                                                int T, int k_side, const uint16_t *__restrict__ v_new,
                                                                uint8_t *__restrict__ v_codes, uint16_t *__restrict__ v_sz,
                                                                uint32_t *__restrict__ v_ptr, const SP vsp, int64_t cap_nnz,
                                                                int32_t *d_status, const KeyCount count)
{
    constexpr int NE = 1 << BITS;
    extern __shared__ __attribute__((aligned(16))) uint4 keys_s[];         // [2 token + quarter][thread]: the keys, for dynamic indices
    __shared__ VpLds lds;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int NT = blockDim.x, nw = NT >> 6;
    if ((int)blockIdx.x < count.wgs) {
        const int t = (int)blockIdx.x * nw + wave;
        if (t < T) k_count_token<true>(params, D, count.k_new, count.cnt, t);
        return;
    }
    const unsigned place = kvq_xcd_place(blockIdx.x - count.wgs, gridDim.x - count.wgs);
    const int64_t m = (n0 >> 1) + place;                                   // the pair
    if (2 * m >= n0 + T) return;
    const int t0 = (int)(2 * m - n0);                                      // the first one's place in the call; -1: not of this call
    const uint32_t own = (t0 >= 0 ? 1u : 0u) | (t0 + 1 < T ? 2u : 0u);     // tokens of the call (a missing one repeats the other)
    const uint32_t K = (uint32_t)k_side;
    const KvqParamsView pv = kvq_params_view(params, D);

    s16x2 s[2][8];
#pragma unroll
    for (int tok = 0; tok < 2; ++tok) {
        const int t = (own >> tok) & 1u ? t0 + tok : t0 + 1 - tok;
        const uint4 *row = (const uint4 *)(v_new + (int64_t)t * D) + 2 * tid;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const uint4 v = row[q];
            s[tok][4 * q] = vp_pair(v.x); s[tok][4 * q + 1] = vp_pair(v.y); s[tok][4 * q + 2] = vp_pair(v.z); s[tok][4 * q + 3] = vp_pair(v.w);
        }
    }
    // thresholds of the codes: lane (token in the lowest bit) looks after one
    const float thr = pv.hdr->thr_v[(lane >> 1) < NE - 1 ? (lane >> 1) : 0];
    const uint32_t first_entry = v_ptr[n0];
    if (tid < 16) lds.lut[tid] = pv.hdr->lut_v[tid & (NE - 1)];
    for (int i = tid; i < 4 * 64; i += NT) (&lds.col_max[0][0])[i] = -32768;
    if (tid < 4) lds.n_cand[tid] = 0;
    if (tid < 3 * KVQ_BULK_MAX_WAVES) (&lds.wave_red[0][0])[tid] = tid < 2 * KVQ_BULK_MAX_WAVES ? 0x80008000u : 0u;
    __syncthreads();
    s16x2 hi[2], lo[2];
#pragma unroll
    for (int tok = 0; tok < 2; ++tok) {
#pragma unroll
        for (int w = 0; w < 8; ++w) s[tok][w] = vp_keys(vp_word(s[tok][w]));
        hi[tok] = lo[tok] = s[tok][0];
#pragma unroll
        for (int w = 1; w < 8; ++w) {
            hi[tok] = __builtin_elementwise_max(hi[tok], s[tok][w]);
            lo[tok] = __builtin_elementwise_min(lo[tok], s[tok][w]);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q)
            keys_s[(2 * tok + q) * NT + tid] = uint4{vp_word(s[tok][4 * q]), vp_word(s[tok][4 * q + 1]), vp_word(s[tok][4 * q + 2]),
                                                     vp_word(s[tok][4 * q + 3])};
    }
    auto key_at = [&](int w, int tok, int half) {        // of this lane
        return (int)((const int16_t *)&keys_s[(2 * tok + (w >> 2)) * NT + tid])[2 * (w & 3) + half];
    };
    uint32_t outl = 0;                                   // outliers: see general_selection
    bool general = false, ties = false;                  // (the same in all wavefronts)
    if (K > 0) {
#pragma unroll
        for (int tok = 0; tok < 2; ++tok) {
            atomicMax(&lds.col_max[2 * tok][lane], (int)(hi[tok].x > hi[tok].y ? hi[tok].x : hi[tok].y));
            atomicMax(&lds.col_max[2 * tok + 1][lane], ~(int)(lo[tok].x < lo[tok].y ? lo[tok].x : lo[tok].y));
        }
        __syncthreads();
        for (int i = wave; i < 4; i += nw) {
            const uint32_t c = (uint32_t)(lds.col_max[i][lane] + 32768);
            uint32_t x = 0;
            for (int bit = 15; bit >= 0; --bit)
                if ((uint32_t)__popcll(__ballot(c >= (x | (1u << bit)))) >= K) x |= 1u << bit;
            if (lane == 0) lds.bound[i] = (int)x - 32768;
        }
        __syncthreads();
        int bound[4];
        uint32_t which = 0;
#pragma unroll
        for (int tok = 0; tok < 2; ++tok) {
            bound[2 * tok] = lds.bound[2 * tok];
            bound[2 * tok + 1] = lds.bound[2 * tok + 1];
            const s16x2 bt = vp_both(bound[2 * tok]), bb = vp_both(~bound[2 * tok + 1]);
#pragma unroll
            for (int w = 0; w < 8; ++w)
                which |= (vp_less(s[tok][w], bt) & vp_less(bb, s[tok][w])) & (0x00010001u << (w + 8 * tok));
        }
        which = ~which;
        int round = 0;
        while (__ballot(which != 0u) != 0ull) {          // (three rounds or so)
            // full lists are of no use: a wavefront stops adding to them (see v_quant_token4)
            if (++round > 4) {
                bool full = false;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    full = full || __hip_atomic_load(&lds.n_cand[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > KVQ_V_CAND;
                if (full) break;
            }
            if (which != 0u) {
                const int b = __ffs((int)which) - 1, tok = (b >> 3) & 1;
                which &= which - 1u;
                const int key = key_at(b & 7, tok, b >> 4);
                const int bt = tok ? bound[2] : bound[0], bb = tok ? bound[3] : bound[1];
                if (key >= bt) {
                    const uint32_t at = atomicAdd(&lds.n_cand[2 * tok], 1u);
                    if (at < KVQ_V_CAND) lds.cand[2 * tok][at] = (uint16_t)(key + 32768);
                }
                if (~key >= bb) {
                    const uint32_t at = atomicAdd(&lds.n_cand[2 * tok + 1], 1u);
                    if (at < KVQ_V_CAND) lds.cand[2 * tok + 1][at] = (uint16_t)(~key + 32768);
                }
            }
        }
        __syncthreads();
        for (int i = wave; i < 4; i += nw) {
            // K-th largest candidate, bit by bit (a list has at least K entries)
            const uint32_t n = lds.n_cand[i];
            uint32_t v[KVQ_V_CAND / 64];
            constexpr int R = KVQ_V_CAND / 64;
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = (uint32_t)lane + 64u * r < n ? lds.cand[i][lane + 64 * r] + 1u : 0u;     // + 1: above an absent one
            auto at_least = [&](uint32_t x) {
                uint32_t c = 0;
#pragma unroll
                for (int r = 0; r < R; ++r) c += (uint32_t)__popcll(__ballot(v[r] >= x));
                return c;
            };
            uint32_t x = 0;
            for (int bit = 16; bit >= 0; --bit)
                if (at_least(x | (1u << bit)) >= K) x |= 1u << bit;
            const uint32_t beyond = at_least(x + 1u), reached = at_least(x);
            if (lane == 0) {
                lds.found[i].tau = (int)x - 1 - 32768;
                lds.found[i].need = K - beyond;
                lds.found[i].n_eq = n <= KVQ_V_CAND ? reached - beyond : ~0u;
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int tau = lds.found[i].tau;
            ties = ties || lds.found[i].need != lds.found[i].n_eq;
            general = general || lds.found[i].n_eq == ~0u || tau == 0 || tau == -1;      // (~0 is -1)
        }
        general = general || lds.found[0].tau == ~lds.found[1].tau || lds.found[2].tau == ~lds.found[3].tau;
        general = __builtin_amdgcn_readfirstlane((int)general) != 0;
        ties = __builtin_amdgcn_readfirstlane((int)ties) != 0 && !general;
        if (general) outl = general_selection(lds, s, K);
    }
    // range of the remaining elements and the number of outliers
    s16x2 mx[2], mn[2];
    if (K == 0) {
#pragma unroll
        for (int tok = 0; tok < 2; ++tok) { mx[tok] = hi[tok]; mn[tok] = lo[tok]; }
    } else if (!general) {
        uint32_t in = 0;
#pragma unroll
        for (int tok = 0; tok < 2; ++tok) {
            const s16x2 tt = vp_both(lds.found[2 * tok].tau), tb = vp_both(~lds.found[2 * tok + 1].tau);
            mx[tok] = vp_both(-32768);
            mn[tok] = vp_both(32767);
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                const uint32_t below = vp_less(s[tok][w], tt), above = vp_less(tb, s[tok][w]);
                // (a lower outlier is no larger than any inlier, of which there is one at least, and the other way round)
                mx[tok] = __builtin_elementwise_max(mx[tok], vp_pair(vp_select(below, vp_word(s[tok][w]), 0x80008000u)));
                mn[tok] = __builtin_elementwise_min(mn[tok], vp_pair(vp_select(above, vp_word(s[tok][w]), 0x7FFF7FFFu)));
                in |= (below & above) & (0x00010001u << (w + 8 * tok));
            }
        }
        outl = ~in;
        if (ties) {
            outl = drop_equals(lds, s, outl);
            // a threshold with equals left over is the extreme of the rest
#pragma unroll
            for (int tok = 0; tok < 2; ++tok) {
                if (lds.found[2 * tok].need < lds.found[2 * tok].n_eq) mx[tok] = vp_both(lds.found[2 * tok].tau);
                if (lds.found[2 * tok + 1].need < lds.found[2 * tok + 1].n_eq) mn[tok] = vp_both(~lds.found[2 * tok + 1].tau);
            }
        }
    } else {
#pragma unroll
        for (int tok = 0; tok < 2; ++tok) {
            mx[tok] = vp_both(-32768);
            mn[tok] = vp_both(32767);
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                const uint32_t o = outl >> (w + 8 * tok);
                const uint32_t out = (o & 1u ? 0xFFFFu : 0u) | ((o >> 16) & 1u ? 0xFFFF0000u : 0u);
                mx[tok] = __builtin_elementwise_max(mx[tok], vp_pair(vp_select(out, 0x80008000u, vp_word(s[tok][w]))));
                mn[tok] = __builtin_elementwise_min(mn[tok], vp_pair(vp_select(out, 0x7FFF7FFFu, vp_word(s[tok][w]))));
            }
        }
    }
    const uint32_t n_out = (uint32_t)__popc(outl & 0x00FF00FFu) | (uint32_t)__popc(outl & 0xFF00FF00u) << 16;
    const uint32_t upto = vp_scan(n_out);
    s16x2 top, bot;                                      // of the tokens: largest inlier, complement of the smallest
    uint32_t before;                                     // outliers of either token before this lane's channels
    auto reduce = [&]() {
        auto larger = [](s16x2 v) { return v.x > v.y ? v.x : v.y; };
        auto smaller = [](s16x2 v) { return v.x < v.y ? v.x : v.y; };
        const s16x2 a = vp_wave_max(s16x2{larger(mx[0]), larger(mx[1])});
        const s16x2 b = vp_wave_max(s16x2{(short)~smaller(mn[0]), (short)~smaller(mn[1])});
        if (lane == 63) { lds.wave_red[0][wave] = vp_word(a); lds.wave_red[1][wave] = vp_word(b); lds.wave_red[2][wave] = upto; }
        __syncthreads();
        uint32_t r[3][8];                                // (wavefronts that there are not: no keys, no outliers)
        static_assert(KVQ_BULK_MAX_WAVES == 8, "two loads");
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const uint4 x = *(const uint4 *)&lds.wave_red[i][0], y = *(const uint4 *)&lds.wave_red[i][4];
            r[i][0] = x.x; r[i][1] = x.y; r[i][2] = x.z; r[i][3] = x.w; r[i][4] = y.x; r[i][5] = y.y; r[i][6] = y.z; r[i][7] = y.w;
        }
        top = bot = vp_both(-32768);
        before = upto - n_out;
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            top = __builtin_elementwise_max(top, vp_pair(r[0][w]));
            bot = __builtin_elementwise_max(bot, vp_pair(r[1][w]));
            before += w < wave ? r[2][w] : 0u;
        }
    };
    reduce();
    constexpr int INF_KEY = 0x7C00;
    const bool nan = top.x > INF_KEY || top.y > INF_KEY || bot.x > INF_KEY || bot.y > INF_KEY;       // among the inliers
    if (nan) {                                           // (the same in all wavefronts) the range is that of the others
        __syncthreads();
#pragma unroll
        for (int tok = 0; tok < 2; ++tok) {
            mx[tok] = vp_both(~INF_KEY);                 // -inf, and inf, where there are none
            mn[tok] = vp_both(INF_KEY);
#pragma unroll 1
            for (int e = 0; e < 16; ++e) {
                const int key = key_at(e >> 1, tok, e & 1);
                if (((outl >> ((e >> 1) + 8 * tok + 16 * (e & 1))) & 1u) || key > INF_KEY || key < ~INF_KEY) continue;
                mx[tok] = __builtin_elementwise_max(mx[tok], vp_both(key));
                mn[tok] = __builtin_elementwise_min(mn[tok], vp_both(key));
            }
        }
        reduce();
    }
    // scale and zero-point: even lanes have the first token's, odd ones the second's
    const float mxf = vp_value((lane & 1) ? top.y : top.x), mnf = vp_value(~(int)((lane & 1) ? bot.y : bot.x));
    const float sum = mxf + mnf, dif = mxf - mnf;
    uint16_t zb = kvq_f2h_rn(sum * 0.5f), sb = kvq_f2h_rn(dif * 0.5f);
    const float zf = kvq_h2f(zb);
    float sf = kvq_h2f(sb);
    if (sf == 0.0f) { sf = 1.0f; sb = 0x3c00u; }
    const float rinv = __fdiv_rn(1.0f, sf);
    const int64_t n = 2 * m;
    if (tid < 2 && ((own >> tid) & 1u)) {
        uint64_t p = (uint64_t)first_entry + (uint32_t)(t0 + tid + 1) * 2u * K;
        if (p > (uint64_t)cap_nnz) { p = (uint64_t)cap_nnz; atomicExch(d_status, (int32_t)KVQ_ERR_NNZ_OVERFLOW); }
        v_ptr[n + tid + 1] = (uint32_t)p;
        v_sz[(n + tid) * 2 + 0] = sb;
        v_sz[(n + tid) * 2 + 1] = zb;
    }
    float z2[2], s2[2], r2[2];
#pragma unroll
    for (int tok = 0; tok < 2; ++tok) {
        z2[tok] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, zf), tok));
        s2[tok] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, sf), tok));
        r2[tok] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, rinv), tok));
    }
    // ---- codes: out[] is this lane's 16 fields (first token's code, second's), 32 BITS bits
    const KvqCoder<NE> coder(pv.hdr->thr_v, pv.hdr->lut_v);
    uint32_t out[BITS] = {};
    auto insert = [&](int w, uint32_t fields) {          // two fields, 4 BITS bits; w a constant
        const int at = 4 * BITS * w, d = at >> 5, sh = at & 31;
        out[d] |= fields << sh;
        if (sh + 4 * BITS > 32) out[d + 1 < BITS ? d + 1 : d] |= fields >> (32 - sh);
    };
    // (normalised inliers lie within [-2, 2] where the scale is finite and not zero)
    const bool plain = !nan && coder.range > 0.0f && s2[0] < INFINITY && s2[1] < INFINITY && __builtin_fabsf(z2[0]) < INFINITY &&
                       __builtin_fabsf(z2[1]) < INFINITY;
    if (plain) {
        const int kj = vp_first_key(thr, sf, zf, rinv);
        const uint32_t twice = ((uint32_t)kj & 0xFFFFu) * 0x10001u;
#pragma unroll
        for (int tok = 0; tok < 2; ++tok) {
            uint32_t k[NE - 1];
#pragma unroll
            for (int j = 0; j < NE - 1; ++j) k[j] = (uint32_t)__builtin_amdgcn_readlane((int)twice, 2 * j + tok);
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                // bit BITS - 1 of the code first; a mask says that the key lies below, so the bits are inverted
                auto bit_at = [&](int v) { return (1u << (tok * BITS + v)) | (1u << (16 + 2 * BITS + tok * BITS + v)); };
                uint32_t fields, l1 = vp_less(s[tok][w], vp_pair(k[NE / 2 - 1])), l2, l3;
                if constexpr (BITS == 2) {
                    l2 = vp_less(s[tok][w], vp_pair(vp_select(l1, k[0], k[2])));
                    fields = (l1 & bit_at(1)) | (l2 & bit_at(0));
                } else if constexpr (BITS == 3) {
                    l2 = vp_less(s[tok][w], vp_pair(vp_select(l1, k[1], k[5])));
                    l3 = vp_less(s[tok][w], vp_pair(vp_select(l2, vp_select(l1, k[0], k[4]), vp_select(l1, k[2], k[6]))));
                    fields = (l1 & bit_at(2)) | (l2 & bit_at(1)) | (l3 & bit_at(0));
                } else {
                    l2 = vp_less(s[tok][w], vp_pair(vp_select(l1, k[3], k[11])));
                    l3 = vp_less(s[tok][w], vp_pair(vp_select(l2, vp_select(l1, k[1], k[9]), vp_select(l1, k[5], k[13]))));
                    const uint32_t a = vp_select(l2, vp_select(l1, k[0], k[8]), vp_select(l1, k[4], k[12]));
                    const uint32_t b = vp_select(l2, vp_select(l1, k[2], k[10]), vp_select(l1, k[6], k[14]));
                    const uint32_t l4 = vp_less(s[tok][w], vp_pair(vp_select(l3, a, b)));
                    fields = (l1 & bit_at(3)) | (l2 & bit_at(2)) | (l3 & bit_at(1)) | (l4 & bit_at(0));
                }
                insert(w, (fields & 0xFFFFu) | (fields >> 16));
            }
        }
#pragma unroll
        for (int d = 0; d < BITS; ++d) out[d] = ~out[d];
    } else {
#pragma unroll 1
        for (int e = 0; e < 16; ++e) {
            uint32_t field = 0;
#pragma unroll
            for (int tok = 0; tok < 2; ++tok)
                field |= (uint32_t)coder((vp_value(key_at(e >> 1, tok, e & 1)) - z2[tok]) * r2[tok]) << (tok * BITS);
            const int at = 2 * BITS * e;
#pragma unroll
            for (int d = 0; d < BITS; ++d) {
                const int sh = at - 32 * d;
                if (sh > -2 * BITS && sh < 32) out[d] |= sh >= 0 ? field << sh : field >> -sh;
            }
        }
    }
    // ---- outliers: the entries, and the codes of those too far out for the thresholds
    bool overflow = false;
    uint32_t left = outl & ((own & 1u ? 0x00FF00FFu : 0u) | (own & 2u ? 0xFF00FF00u : 0u));
    while (__ballot(left != 0u) != 0ull) {
        if (left == 0u) continue;
        const int b = __ffs((int)left) - 1, w = b & 7, tok = (b >> 3) & 1, half = b >> 4;
        left &= left - 1u;
        const float x = vp_value(key_at(w, tok, half));
        const float z = tok ? z2[1] : z2[0], sc = tok ? s2[1] : s2[0], ri = tok ? r2[1] : r2[0];
        const float diff = x - z, xn = diff * ri;
        int code = coder.count(xn);
        if (plain && coder.far(xn)) {
            code = coder.search(xn);
            const int at = 2 * BITS * (2 * w + half) + BITS * tok;
#pragma unroll
            for (int d = 0; d < BITS; ++d) {
                const int sh = at - 32 * d;
                if (sh > -BITS && sh < 32) {
                    const uint32_t mask = sh >= 0 ? (uint32_t)(NE - 1) << sh : (uint32_t)(NE - 1) >> -sh;
                    out[d] = (out[d] & ~mask) | (sh >= 0 ? (uint32_t)code << sh : (uint32_t)code >> -sh);
                }
            }
        } else if (!plain) {
            code = coder(xn);
        }
        const uint32_t lower = ((1u << w) - 1u) * 0x00010001u | (half ? 1u << w : 0u);        // this lane's channels below
        const uint32_t rank = ((before >> (16 * tok)) & 0xFFFFu) + (uint32_t)__popc(outl & (lower << (8 * tok)));
        const uint64_t pos = (uint64_t)first_entry + (uint32_t)(t0 + tok) * 2u * K + rank;
        if (pos < (uint64_t)cap_nnz) vsp.put(pos, (uint16_t)(16 * tid + 2 * w + half), kvq_f2h_rn(x - __builtin_fmaf(sc, lds.lut[code], z)));
        else overflow = true;
    }
    if (overflow) atomicExch(d_status, (int32_t)KVQ_ERR_NNZ_OVERFLOW);
    // ---- store: dwords (tid & 3) BITS .. + BITS - 1 of the chunk of 64 channels
    uint8_t *chunk = v_codes + kvq_v_piece0(BITS, cap, m, tid >> 3, (tid >> 2) & 1);
    if (own == 3u) {
        const int d = (tid & 3) * BITS;
        uint8_t *p = chunk + (d >> 2) * 1024 + (d & 3) * 4;
        if constexpr (BITS == 4) {
            *(uint4 *)p = uint4{out[0], out[1], out[2], out[3]};
        } else if constexpr (BITS == 2) {
            *(uint2 *)p = uint2{out[0], out[1]};
        } else {
#pragma unroll
            for (int i = 0; i < BITS; ++i) *(uint32_t *)(chunk + ((d + i) >> 2) * 1024 + ((d + i) & 3) * 4) = out[i];
        }
    } else {
        // one token: the other bits of the dwords belong to its partner
        const int parity = own == 2u ? 1 : 0;
#pragma unroll
        for (int i = 0; i < BITS; ++i) {
            uint32_t mask = 0;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int sh = 2 * BITS * e - 32 * i;                      // of the field; the partner's half of it is the other one
                const uint32_t f = (uint32_t)(NE - 1) << (parity * BITS);
                if (sh > -2 * BITS && sh < 32) mask |= sh >= 0 ? f << sh : f >> -sh;
            }
            const int d = (tid & 3) * BITS + i;
            uint32_t *p = (uint32_t *)(chunk + (d >> 2) * 1024 + (d & 3) * 4);
            __hip_atomic_fetch_and(p, ~mask, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_or(p, out[i] & mask, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

}  // namespace

void kvq_v_pair_launch(const kvq_cache *c, const uint16_t *d_v_new, int T, unsigned pairs, int count_wgs, const uint16_t *k_new,
                       uint32_t *k_count, hipStream_t s)
{
    const int D = c->n_kv_heads * KVQ_HEAD_DIM;
    count_wgs = (int)kvq_xcd_grid(count_wgs);            // (the pairs' places count from a multiple of eight)
    const KeyCount count = {count_wgs, k_new, k_count};
    const auto launch = [&](auto bits, const auto vsp) {
        kvq_v_pair<decltype(bits)::value><<<kvq_xcd_grid(pairs) + count_wgs, D / 16, 4 * D, s>>>(
            c->params, D, c->cap_tokens, c->n_tokens_v, T, c->k_side_v, d_v_new, c->v_codes, c->v_sz, c->v_ptr, vsp, c->cap_nnz_v,
            c->d_status, count);
    };
    const auto by_bits = [&](const auto vsp) {
        if (c->bits == 2) launch(std::integral_constant<int, 2>{}, vsp);
        else if (c->bits == 3) launch(std::integral_constant<int, 3>{}, vsp);
        else launch(std::integral_constant<int, 4>{}, vsp);
    };
    if (c->nnz_block_shift) by_bits(kvq_blocked_v(c));
    else by_bits(kvq_flat_v(c));
}
