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
//    keys on and beyond the bounds are collected and the thresholds found among them with ballots -, but each of the four searches
//    (two tokens, two sides) by one wavefront for all, and one list for both sides of a token;
//  * codes: the normalised value grows with x, so that the code of x is the number of keys K_j <= x where K_j is the smallest
//    fp16 number whose normalised value (the same fp32 steps) reaches the j-th threshold.  One lane per threshold and token
//    finds its K_j, next to where the inverse of the normalisation points; an element's code is a binary search of
//    log2 comparisons, each a saturating subtraction whose sign selects the next K_j.
//  * outliers: their channels go to a list by rank, and a lane takes any of them, so that outliers crowded in few lanes' channels
//    do not take longer; codes beyond the code range are put right by the lanes that hold them.
// Where more keys than a list holds lie on and beyond the bounds, those beyond alone are listed (crowds of equal keys, zeros above all: with fewer than
// k beyond, the bound is the threshold); then the same with other columns (the largest keys in few lanes), at last a bisection over all keys.
// Where only some of a threshold's equals are outliers, they are ranked in channel order.  Same arithmetic, same results, as v_quant_token.
// us per Value append, the kernel with a token on four wavefronts and a lane per element (v_quant_token4) / this one, 1 % outliers:
// 4096 tokens of 4096 channels, 2 bits 46.5 / 22.5, 3 bits 50.9 / 25.1, 4 bits 56.5 / 27.9; of 5120, 4 bits 77.3 / 41.4; of 8192, 3 bits 107 / 47; 777 of
// 5120, 4 bits, 22.9 / 14.2; 64 of 4096 14.3 / 9.0; 4096 of 3072 (the routine for any width before) 81.6 / 21.2.  4096 tokens of 4096 channels, 3 bits, that are
// ordinary 50.9 / 25.1, zero 99 / 41, zero or positive 104 / 38, every third zero 78 / 37, with one head eight times as large 48 / 33, sixteen channels 50 / 35, but
// sorted 46 / 62.  Bound by vector issue, with six wavefronts a SIMD, 80 registers and no spills (eight, which spilled: 4096 channels slower by 4 %).

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
// Zeros of both signs are one key, 0, to them.
constexpr int VP_CAND = 512;                     // candidates of a token that a list holds
struct VpLds {
    union {
        int col_max[4][64];                    // the largest keys of the 64 columns (lane l of every wavefront)
        uint16_t cand[2][VP_CAND];             // candidates of either side, + 32768
    };
    uint32_t n_cand[2], n_side[2];             // tokens packed: candidates on and beyond the bounds, beyond them; by side, those beyond
    int bound[4];                              // keys
    struct { int tau; uint32_t need, n_eq; } found[4];     // threshold, a key; how many of its equals are taken, how many there are (~0: not known)
    __attribute__((aligned(16))) uint32_t wave_red[3][KVQ_BULK_MAX_WAVES];       // of a wavefront's inliers (tokens packed): largest, complement of smallest; outliers
    uint32_t counts[17][2];                    // general_selection's rounds
    uint32_t eq[KVQ_BULK_MAX_WAVES][2];
    uint16_t ids[2][2 * KVQ_V_BOUNDED];        // channels of the outliers
    float lut[16];
};
// The smallest key that equals a threshold.
__device__ __forceinline__ int vp_least_equal(int tau) { return tau == 0 ? -1 : tau; }

// Of search i: the k-th largest among its token's n candidates, K <= n <= 64 R, bit by bit.  (Those of the other side change nothing.)
template <int R>
__device__ __forceinline__ void pick(VpLds &lds, int i, uint32_t n, uint32_t K)
{
    const int lane = threadIdx.x & 63;
    const uint16_t *list = lds.cand[i >> 1];
    uint32_t v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t u = list[lane + 64 * r];
        v[r] = (uint32_t)lane + 64u * r < n ? ((i & 1) ? 65536u - u : u + 1u) : 0u;        // (above an absent one)
    }
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
        lds.found[i].tau = ((i & 1) ? (int)(65536u - x) : (int)x - 1) - 32768;
        lds.found[i].need = K - beyond;
        lds.found[i].n_eq = reached - beyond;
    }
}

// This lane's column where lanes do not serve: groups of four channels that lie a multiple of 256 apart, of a wavefront's channels.  Half of a
// wavefront's words are exchanged for the other half's, then a row's for its neighbour's: packed extremes of either fall on one lane.
__device__ __forceinline__ void vp_column_of_fours(const s16x2 (&s)[8], s16x2 &most, s16x2 &least)
{
    s16x2 mx[4], mn[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const auto r = __builtin_amdgcn_permlane32_swap(vp_word(s[j]), vp_word(s[j + 4]), false, false);
        mx[j] = __builtin_elementwise_max(vp_pair(r[0]), vp_pair(r[1]));
        mn[j] = __builtin_elementwise_min(vp_pair(r[0]), vp_pair(r[1]));
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const auto a = __builtin_amdgcn_permlane16_swap(vp_word(mx[j]), vp_word(mx[j + 2]), false, false);
        const auto b = __builtin_amdgcn_permlane16_swap(vp_word(mn[j]), vp_word(mn[j + 2]), false, false);
        mx[j] = __builtin_elementwise_max(vp_pair(a[0]), vp_pair(a[1]));
        mn[j] = __builtin_elementwise_min(vp_pair(b[0]), vp_pair(b[1]));
    }
    most = __builtin_elementwise_max(mx[0], mx[1]);
    least = __builtin_elementwise_min(mn[0], mn[1]);
}

// The thresholds of both tokens where the lists do not serve either: by bisection over all keys, a barrier a bit.
__device__ __forceinline__ void general_selection(VpLds &lds, const s16x2 (&s)[2][8], uint32_t K)
{
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid; i < 17 * 2; i += blockDim.x) (&lds.counts[0][0])[i] = 0;
    __syncthreads();
    uint32_t x[4] = {0, 0, 0, 0};                        // (of larger keys, and on side 1 of smaller ones)
#pragma unroll 1
    for (int bit = 15; bit >= -1; --bit) {               // (the last round: how many exceed the thresholds themselves)
#pragma unroll
        for (int tok = 0; tok < 2; ++tok) {
            // keys above a and below b
            int a, b;
            if (bit >= 0) {
                a = vp_least_equal((int)(x[2 * tok] | (1u << bit)) - 32768) - 1;
                b = 32767 - (int)(x[2 * tok + 1] | (1u << bit));
                b = b == -1 ? -1 : b + 1;
            } else {
                a = (int)x[2 * tok] - 32768;
                b = vp_least_equal(32767 - (int)x[2 * tok + 1]);
            }
            const s16x2 va = vp_both(a), vb = vp_both(b);
            s16x2 above = {0, 0}, below = {0, 0};        // less their numbers
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                above += vp_pair(vp_less(va, s[tok][w]));
                below += vp_pair(vp_less(s[tok][w], vb));
            }
            const uint32_t n = (uint32_t)-(above.x + above.y) | (uint32_t)-(below.x + below.y) << 16;
            const uint32_t sum = (uint32_t)__builtin_amdgcn_readlane((int)vp_scan(n), 63);
            if (lane == 0) atomicAdd(&lds.counts[15 - bit][tok], sum);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t n = (lds.counts[15 - bit][i >> 1] >> (16 * (i & 1))) & 0xFFFFu;
            if (bit >= 0) {
                if (n >= K) x[i] |= 1u << bit;
            } else if (tid == 0) {
                lds.found[i].tau = (i & 1) ? 32767 - (int)x[i] : (int)x[i] - 32768;
                lds.found[i].need = K - n;
                lds.found[i].n_eq = ~0u;
            }
        }
    }
}

// The outliers where only some of a threshold's equals are: the keys beyond, and of the equals the first in channel order.
__device__ __forceinline__ uint32_t with_equals(VpLds &lds, const s16x2 (&s)[2][8])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t outl = 0, eq[2] = {0, 0}, before[2];        // by side
#pragma unroll
    for (int tok = 0; tok < 2; ++tok) {
        const int top = lds.found[2 * tok].tau, bot = lds.found[2 * tok + 1].tau;
        const s16x2 t = vp_both(top), t0 = vp_both(vp_least_equal(top)), b = vp_both(bot), b0 = vp_both(vp_least_equal(bot));
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const uint32_t bits = 0x00010001u << (w + 8 * tok), above = vp_less(t, s[tok][w]), below = vp_less(s[tok][w], b0);
            outl |= (above | below) & bits;
            eq[0] |= ~(above | vp_less(s[tok][w], t0)) & bits;
            eq[1] |= ~(below | vp_less(b, s[tok][w])) & bits;
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
            // equals from rank `from` to `to`; thresholds coincide: the lower outliers take those that follow the upper ones'
            const bool same = lds.found[2 * tok].tau == lds.found[2 * tok + 1].tau;
            const uint32_t from = side && same ? lds.found[2 * tok].need : 0u, to = from + lds.found[2 * tok + side].need;
            uint32_t rank = (before[side] >> (16 * tok)) & 0xFFFFu, left = (eq[side] >> (8 * tok)) & 0x00FF00FFu;
            const uint32_t end = rank + (uint32_t)__popc(left);
            if (rank >= from && end <= to) {             // all of them, or none: nearly every lane
                outl |= left << (8 * tok);
            } else if (rank < to && end > from) {
                while (left != 0u) {                     // in channel order: words, then halves
                    const int w = __ffs((int)((left | left >> 16) & 0xFFu)) - 1;
                    const uint32_t bit = 1u << w & left ? 1u << w : 0x10000u << w;
                    left &= ~bit;
                    if (rank >= from && rank < to) outl |= bit << (8 * tok);
                    ++rank;
                }
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
    if (tid < 2) lds.n_cand[tid] = lds.n_side[tid] = 0;
    if (tid < 3 * KVQ_BULK_MAX_WAVES) (&lds.wave_red[0][0])[tid] = tid < 2 * KVQ_BULK_MAX_WAVES ? 0x80008000u : 0u;
    __syncthreads();
    auto extremes = [&](int tok, s16x2 &most, s16x2 &least) {              // of this lane
        most = least = s[tok][0];
#pragma unroll
        for (int w = 1; w < 8; ++w) {
            most = __builtin_elementwise_max(most, s[tok][w]);
            least = __builtin_elementwise_min(least, s[tok][w]);
        }
    };
#pragma unroll
    for (int tok = 0; tok < 2; ++tok) {
#pragma unroll
        for (int w = 0; w < 8; ++w) s[tok][w] = vp_keys(vp_word(s[tok][w]));
#pragma unroll
        for (int q = 0; q < 2; ++q)
            keys_s[(2 * tok + q) * NT + tid] = uint4{vp_word(s[tok][4 * q]), vp_word(s[tok][4 * q + 1]), vp_word(s[tok][4 * q + 2]),
                                                     vp_word(s[tok][4 * q + 3])};
    }
    auto key_at = [&](int w, int tok, int half) {        // of this lane
        return (int)((const int16_t *)&keys_s[(2 * tok + (w >> 2)) * NT + tid])[2 * (w & 3) + half];
    };
    uint32_t outl = 0;                                   // outliers: bit w + 8 token + 16 half is half `half` of this lane's word w
    bool ties = false;                                   // (the same in all wavefronts)
    if (K > 0) {
        // Keys go to the token's list, a run of places for each wavefront's; none, if there are more than it holds.
        auto collect = [&](uint32_t which, uint32_t *count) {
            const uint32_t mine = (uint32_t)__popc(which & 0x00FF00FFu) | (uint32_t)__popc(which & 0xFF00FF00u) << 16, upto = vp_scan(mine);
            uint32_t at = 0;
            if (lane == 63) at = atomicAdd(count, upto);
            at = (uint32_t)__builtin_amdgcn_readlane((int)at, 63);
            const uint32_t end = at + (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
            if ((end & 0xFFFFu) > (uint32_t)VP_CAND || end >> 16 > (uint32_t)VP_CAND) return;
            at += upto - mine;
            while (__ballot(which != 0u) != 0ull) {      // (two or three rounds)
                if (which == 0u) continue;
                const int b = __ffs((int)which) - 1, tok = (b >> 3) & 1;
                which &= which - 1u;
                const int key = key_at(b & 7, tok, b >> 4);
                lds.cand[tok][tok ? at >> 16 : at & 0xFFFFu] = (uint16_t)((key == -1 ? 0 : key) + 32768);
                at += tok ? 0x10000u : 1u;
            }
        };
        auto full = [](uint32_t n) { return (n & 0xFFFFu) > (uint32_t)VP_CAND || n >> 16 > (uint32_t)VP_CAND; };
        uint32_t n_cand;
        bool crowd, general;
#pragma unroll 1
        for (int attempt = 0;; ++attempt) {
#pragma unroll
            for (int tok = 0; tok < 2; ++tok) {
                s16x2 hi, lo;
                if (attempt == 0) extremes(tok, hi, lo);
                else vp_column_of_fours(s[tok], hi, lo);
                atomicMax(&lds.col_max[2 * tok][lane], (int)(hi.x > hi.y ? hi.x : hi.y));
                atomicMax(&lds.col_max[2 * tok + 1][lane], ~(int)(lo.x < lo.y ? lo.x : lo.y));
            }
            __syncthreads();
            for (int i = wave; i < 4; i += nw) {
                const uint32_t c = (uint32_t)(lds.col_max[i][lane] + 32768);
                uint32_t x = 0;
                for (int bit = 15; bit >= 0; --bit)
                    if ((uint32_t)__popcll(__ballot(c >= (x | (1u << bit)))) >= K) x |= 1u << bit;
                const int b = (i & 1) ? ~((int)x - 32768) : (int)x - 32768;
                if (lane == 0) lds.bound[i] = b == -1 ? 0 : b;
            }
            __syncthreads();
            uint32_t which = 0;
#pragma unroll
            for (int tok = 0; tok < 2; ++tok) {
                const s16x2 t0 = vp_both(vp_least_equal(lds.bound[2 * tok])), b = vp_both(lds.bound[2 * tok + 1]);
#pragma unroll
                for (int w = 0; w < 8; ++w) which |= (vp_less(s[tok][w], t0) & vp_less(b, s[tok][w])) & (0x00010001u << (w + 8 * tok));
            }
            collect(~which, &lds.n_cand[0]);
            __syncthreads();
            n_cand = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds.n_cand[0]);
            crowd = full(n_cand);
            general = false;
            if (crowd) {
                // Many keys on a bound: those beyond are listed.  Where they are fewer than K, the bound is the threshold.
                uint32_t beyond[2] = {0, 0};
#pragma unroll
                for (int tok = 0; tok < 2; ++tok) {
                    const s16x2 t = vp_both(lds.bound[2 * tok]), b0 = vp_both(vp_least_equal(lds.bound[2 * tok + 1]));
#pragma unroll
                    for (int w = 0; w < 8; ++w) {
                        beyond[0] |= vp_less(t, s[tok][w]) & (0x00010001u << (w + 8 * tok));
                        beyond[1] |= vp_less(s[tok][w], b0) & (0x00010001u << (w + 8 * tok));
                    }
                }
#pragma unroll
                for (int side = 0; side < 2; ++side) {
                    const uint32_t upto = vp_scan((uint32_t)__popc(beyond[side] & 0x00FF00FFu) | (uint32_t)__popc(beyond[side] & 0xFF00FF00u) << 16);
                    if (lane == 63) atomicAdd(&lds.n_side[side], upto);
                }
                collect(beyond[0] | beyond[1], &lds.n_cand[1]);
                __syncthreads();
                n_cand = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds.n_cand[1]);
                general = full(n_cand);
            }
            if (!general || attempt == 1) break;
            // the largest keys in few lanes: once more with other columns
            for (int i = tid; i < 4 * 64; i += NT) (&lds.col_max[0][0])[i] = -32768;
            __syncthreads();
            if (tid < 2) lds.n_cand[tid] = lds.n_side[tid] = 0;
        }
        if (general) {
            general_selection(lds, s, K);
        } else {
            for (int i = wave; i < 4; i += nw) {
                const uint32_t n = (n_cand >> (16 * (i >> 1))) & 0xFFFFu;
                const uint32_t beyond = crowd ? (lds.n_side[i & 1] >> (16 * (i >> 1))) & 0xFFFFu : K;
                if (beyond < K) {
                    if (lane == 0) { lds.found[i].tau = lds.bound[i]; lds.found[i].need = K - beyond; lds.found[i].n_eq = ~0u; }
                } else if (n <= 64u) {
                    pick<1>(lds, i, n, K);
                } else if (n <= 128u) {
                    pick<2>(lds, i, n, K);
                } else if (n <= 192u) {
                    pick<3>(lds, i, n, K);
                } else {
                    pick<VP_CAND / 64>(lds, i, n, K);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) ties = ties || lds.found[i].need != lds.found[i].n_eq;
        ties = ties || lds.found[0].tau == lds.found[1].tau || lds.found[2].tau == lds.found[3].tau;
        ties = __builtin_amdgcn_readfirstlane((int)ties) != 0;
        if (ties) outl = with_equals(lds, s);
    }
    // range of the remaining elements and the number of outliers
    s16x2 mx[2], mn[2];
    if (K == 0) {
#pragma unroll
        for (int tok = 0; tok < 2; ++tok) extremes(tok, mx[tok], mn[tok]);
    } else if (!ties) {
        uint32_t in = 0;
#pragma unroll
        for (int tok = 0; tok < 2; ++tok) {
            const s16x2 tt = vp_both(vp_least_equal(lds.found[2 * tok].tau)), tb = vp_both(lds.found[2 * tok + 1].tau);
            mx[tok] = vp_both(-32768);
            mn[tok] = vp_both(32767);
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                const uint32_t below = vp_less(s[tok][w], tt), above = vp_less(tb, s[tok][w]);
                // (a lower outlier is less than any inlier, of which there is one at least, and the other way round)
                mx[tok] = __builtin_elementwise_max(mx[tok], vp_pair(vp_select(below, vp_word(s[tok][w]), 0x80008000u)));
                mn[tok] = __builtin_elementwise_min(mn[tok], vp_pair(vp_select(above, vp_word(s[tok][w]), 0x7FFF7FFFu)));
                in |= (below & above) & (0x00010001u << (w + 8 * tok));
            }
        }
        outl = ~in;
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
    // ---- outliers: a wavefront's channels into a list by their places among the token's, then an entry to a lane, whichever lanes they
    // came from
    bool overflow = false;
    {
        uint32_t left = outl & ((own & 1u ? 0x00FF00FFu : 0u) | (own & 2u ? 0xFF00FF00u : 0u));
        while (__ballot(left != 0u) != 0ull) {
            if (left == 0u) continue;
            const int b = __ffs((int)left) - 1, w = b & 7, tok = (b >> 3) & 1, half = b >> 4;
            left &= left - 1u;
            const uint32_t lower = ((1u << w) - 1u) * 0x00010001u | (half ? 1u << w : 0u);    // this lane's channels below
            const uint32_t rank = ((before >> (16 * tok)) & 0xFFFFu) + (uint32_t)__popc(outl & (lower << (8 * tok)));
            if (rank < 2u * KVQ_V_BOUNDED) lds.ids[tok][rank] = (uint16_t)(16 * tid + 2 * w + half);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    const uint32_t first_rank = (uint32_t)__builtin_amdgcn_readfirstlane((int)before);
    const uint32_t here = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
    const int here0 = own & 1u ? (int)(here & 0xFFFFu) : 0, here1 = own & 2u ? (int)(here >> 16) : 0;
    bool any_far = false;
    for (int e = lane; __ballot(e < here0 + here1) != 0ull; e += 64) {
        bool far = false;
        if (e < here0 + here1) {
            const int tok = e >= here0 ? 1 : 0;
            const uint32_t rank = ((first_rank >> (16 * tok)) & 0xFFFFu) + (uint32_t)(tok ? e - here0 : e);
            const uint32_t c = lds.ids[tok][rank];
            const float x = vp_value((int)((const int16_t *)&keys_s[(2 * tok + ((c >> 3) & 1)) * NT + (c >> 4)])[c & 7]);
            const float z = tok ? z2[1] : z2[0], sc = tok ? s2[1] : s2[0], ri = tok ? r2[1] : r2[0];
            const float diff = x - z, xn = diff * ri;
            far = coder.far(xn);
            const int code = far ? coder.search(xn) : coder.count(xn);
            const uint64_t pos = (uint64_t)first_entry + (uint32_t)(t0 + tok) * 2u * K + rank;
            if (pos < (uint64_t)cap_nnz) vsp.put(pos, (uint16_t)c, kvq_f2h_rn(x - __builtin_fmaf(sc, lds.lut[code], z)));
            else overflow = true;
        }
        any_far = any_far || __ballot(far) != 0ull;
    }
    if (plain && any_far) {                              // codes of those too far out for the thresholds
        uint32_t left = outl;
        while (__ballot(left != 0u) != 0ull) {
            if (left == 0u) continue;
            const int b = __ffs((int)left) - 1, w = b & 7, tok = (b >> 3) & 1, half = b >> 4;
            left &= left - 1u;
            const float xn = (vp_value(key_at(w, tok, half)) - (tok ? z2[1] : z2[0])) * (tok ? r2[1] : r2[0]);
            if (!coder.far(xn)) continue;
            const int code = coder.search(xn), at = 2 * BITS * (2 * w + half) + BITS * tok;
#pragma unroll
            for (int d = 0; d < BITS; ++d) {
                const int sh = at - 32 * d;
                if (sh > -BITS && sh < 32) {
                    const uint32_t mask = sh >= 0 ? (uint32_t)(NE - 1) << sh : (uint32_t)(NE - 1) >> -sh;
                    out[d] = (out[d] & ~mask) | (sh >= 0 ? (uint32_t)code << sh : (uint32_t)code >> -sh);
                }
            }
        }
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
