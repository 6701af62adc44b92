// Bulk Key append, a workgroup per run of tokens: lane l of a head's eight has channels 8 l .. 8 l + 7 and the eight 64 further up, the
// ones they share fields with, so a lane's fields are a run of the head's chunk, and the workgroup one thread per sixteen channels
// (D a multiple of 1024).  As in kvq_v_pair.hip elements are signed 16-bit keys, two to a register; here a channel's code thresholds do not
// depend on the token: kvq_lut_load leaves the smallest fp16 number that reaches each (KvqKeyParams), and a lane loads its
// channels' once for all tokens of the run.  The same for the range beyond which an element is an outlier, or so far out that its code
// has to be searched for.
// Pointers: a workgroup adds up the outlier counts of the tokens before its run (kvq_k_count) for itself, instead of a launch between.
// Same arithmetic, same results, as k_quant_token.
// us per Key append, a wavefront per token and a lane per element (kvq_k_quant_wave) / this one, the counts of 7 us included, 1 % outliers: 4096 tokens
// of 4096 channels, 2 bits 36.6 / 24.4, 3 bits 39.7 / 27.3, 4 bits 46.3 / 32.9.  Of the 20 us of the 3-bit kernel nine are the bytes, the rest vector
// issue and the latency of a token's chain (load, ranks over a barrier, outliers one by one) at four wavefronts a SIMD.  What it took: the channels'
// constants loaded at once and not in a loop (-4 us); neighbouring runs on one XCD (-3 %).
#include <type_traits>
#include "kvq_append_common.hpp"
#include "kvq_append_keys.hpp"

namespace {

template <int BITS, class SP>
__global__ __launch_bounds__(64 * KVQ_BULK_MAX_WAVES) void kvq_k_bulk(const void *__restrict__ params, int D, int64_t cap, int64_t n0,
                                                                      int T, int run, const uint16_t *__restrict__ k_new,
                                                                      const uint32_t *__restrict__ cnt, uint8_t *__restrict__ k_codes,
                                                                      uint32_t *__restrict__ k_ptr, const SP ksp, int64_t cap_nnz,
                                                                      int32_t *d_status)
{
    constexpr int NE = 1 << BITS;
    // [thread], what a lane keeps for a dynamic index: 2 the token's keys, 2 its channels' scales, 2 their zero-points
    extern __shared__ __attribute__((aligned(16))) uint4 bulk_s[];
    __shared__ float lut_s[16];
    __shared__ __attribute__((aligned(16))) uint32_t wave_sum[2][KVQ_BULK_MAX_WAVES];      // (none: 0)
    __shared__ uint32_t before_s[KVQ_BULK_MAX_WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int NT = blockDim.x, nw = NT >> 6;
    const KvqParamsView pv = kvq_params_view(params, D);
    const KvqKeyParams kp = kvq_key_params(params, D);
    const int ta = (int)kvq_xcd_place(blockIdx.x, gridDim.x) * run, tb = ta + run < T ? ta + run : T;
    if (ta >= T) return;
    const int h = tid >> 3, l8 = tid & 7, c0 = h * KVQ_HEAD_DIM + 8 * l8;  // lower channels; the upper ones 64 further
    auto words = [](const uint4 &v, uint32_t (&w)[4]) { w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w; };
    auto load = [&](int t, uint32_t (&w)[8]) {
        const uint4 a = *(const uint4 *)(k_new + (int64_t)t * D + c0), b = *(const uint4 *)(k_new + (int64_t)t * D + c0 + 64);
        w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w;
        w[4] = b.x; w[5] = b.y; w[6] = b.z; w[7] = b.w;
    };
    uint32_t next[8];
    load(ta, next);
    // this lane's channels: thresholds of the codes, range of the elements that need nothing else, channels where that range ends
    // before the outliers begin
    uint32_t thr[NE - 1][8], first[8], last[8];
#pragma unroll
    for (int z = 0; z < 2; ++z) {
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < NE - 1; ++j) {
            words(*(const uint4 *)(kp.thr + (int64_t)j * D + c0 + 64 * z), w);
#pragma unroll
            for (int i = 0; i < 4; ++i) thr[j][4 * z + i] = w[i];
        }
        words(*(const uint4 *)(kp.first + c0 + 64 * z), w);
#pragma unroll
        for (int i = 0; i < 4; ++i) first[4 * z + i] = w[i];
        words(*(const uint4 *)(kp.last + c0 + 64 * z), w);
#pragma unroll
        for (int i = 0; i < 4; ++i) last[4 * z + i] = w[i];
    }
    const bool narrow = kp.narrow[c0 >> 3] != 0 || kp.narrow[(c0 + 64) >> 3] != 0;
#pragma unroll
    for (int z = 0; z < 2; ++z) {
        bulk_s[(2 + z) * NT + tid] = *(const uint4 *)(pv.s16 + c0 + 64 * z);
        bulk_s[(4 + z) * NT + tid] = *(const uint4 *)(pv.z16 + c0 + 64 * z);
    }
    if (tid < 2 * KVQ_BULK_MAX_WAVES) (&wave_sum[0][0])[tid] = 0;
    if (tid < 16) lut_s[tid] = pv.hdr->lut_k[tid & (NE - 1)];
    const bool countable = pv.hdr->thr_k[0] == pv.hdr->thr_k[0];
    // outliers of the tokens before the run
    uint32_t sum = 0;
    for (int t4 = 4 * tid; t4 < ta; t4 += 16 * NT) {
        uint4 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = *(const uint4 *)(cnt + (t4 + 4 * i * NT < ta ? t4 + 4 * i * NT : t4));     // (whole groups of four)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int t = t4 + 4 * i * NT;
            sum += (t < ta ? v[i].x : 0u) + (t + 1 < ta ? v[i].y : 0u) + (t + 2 < ta ? v[i].z : 0u) + (t + 3 < ta ? v[i].w : 0u);
        }
    }
    sum = vp_scan(sum);
    if (lane == 63) before_s[wave] = sum;
    const uint32_t ptr0 = k_ptr[n0];
    __syncthreads();
    uint64_t base = ptr0;                                                  // first entry of the token
    for (int w = 0; w < nw; ++w) base += before_s[w];
    bool overflow = false;
    for (int t = ta; t < tb; ++t) {
        s16x2 s[8];
        half2_t odd = {(half_t)0, (half_t)0};                              // NaN: one of the elements is
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            odd = __builtin_elementwise_maximum(odd, __builtin_bit_cast(half2_t, next[i]));
            s[i] = vp_keys(next[i]);
        }
        if (t + 1 < tb) load(t + 1, next);
        bulk_s[tid] = uint4{vp_word(s[0]), vp_word(s[1]), vp_word(s[2]), vp_word(s[3])};
        bulk_s[NT + tid] = uint4{vp_word(s[4]), vp_word(s[5]), vp_word(s[6]), vp_word(s[7])};
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");             // (read by this lane only)
        auto key_at = [&](int w, int half) { return (int)((const int16_t *)&bulk_s[(w >> 2) * NT + tid])[2 * (w & 3) + half]; };
        uint32_t nan = 0;                                                  // no outliers, code 0: below every threshold from here on
        if (__ballot(!(odd.x == odd.x) || !(odd.y == odd.y)) != 0ull) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t m = vp_less(vp_both(31744), s[i]) | vp_less(s[i], vp_both(-31745));
                nan |= m & (0x00010001u << i);
                s[i] = vp_pair(vp_select(m, 0x80008000u, vp_word(s[i])));
            }
        }
        // outliers: bit w + 16 half is half `half` of word w
        uint32_t in = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) in |= ~(vp_less(s[i], vp_pair(first[i])) | vp_less(vp_pair(last[i]), s[i])) & (0x00010001u << i);
        uint32_t outl = ~(in | nan) & 0x00FF00FFu;
        // fields: 16 BITS bits from the lowest on; a mask says that the key lies below a threshold, so the bits are inverted at first
        uint64_t out = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t fields = 0;
#pragma unroll
            for (int z = 0; z < 2; ++z) {
                const s16x2 x = s[4 * z + i];
                auto k = [&](int j) { return thr[j][4 * z + i]; };
                auto below = [&](uint32_t th) { return vp_less(x, vp_pair(th)); };
                auto bit = [&](int v) { return (1u << (z * BITS + v)) | (1u << (16 + 2 * BITS + z * BITS + v)); };
                const uint32_t l1 = below(k(NE / 2 - 1));
                if constexpr (BITS == 2) {
                    fields |= (l1 & bit(1)) | (below(vp_select(l1, k(0), k(2))) & bit(0));
                } else if constexpr (BITS == 3) {
                    const uint32_t l2 = below(vp_select(l1, k(1), k(5)));
                    const uint32_t l3 = below(vp_select(l2, vp_select(l1, k(0), k(4)), vp_select(l1, k(2), k(6))));
                    fields |= (l1 & bit(2)) | (l2 & bit(1)) | (l3 & bit(0));
                } else {
                    const uint32_t l2 = below(vp_select(l1, k(3), k(11)));
                    const uint32_t l3 = below(vp_select(l2, vp_select(l1, k(1), k(9)), vp_select(l1, k(5), k(13))));
                    const uint32_t a = vp_select(l2, vp_select(l1, k(0), k(8)), vp_select(l1, k(4), k(12)));
                    const uint32_t b = vp_select(l2, vp_select(l1, k(2), k(10)), vp_select(l1, k(6), k(14)));
                    fields |= (l1 & bit(3)) | (l2 & bit(2)) | (l3 & bit(1)) | (below(vp_select(l3, a, b)) & bit(0));
                }
            }
            out |= (uint64_t)((fields & 0xFFFFu) | (fields >> 16)) << (4 * BITS * i);
        }
        out = ~out;
        // (an infinity is an outlier like another: a channel whose threshold it does not pass has a range that ends before)
        const bool check = !countable || (narrow && outl != 0u);
        if (__ballot(check) != 0ull) {
            if (check) {                                                   // one by one
                const KvqCoder<NE> coder(pv.hdr->thr_k, pv.hdr->lut_k);
                outl = 0;
                out = 0;
#pragma unroll 1
                for (int e = 0; e < 16; ++e) {
                    const int w = e & 7, half = e >> 3, c = c0 + (w >> 2) * 64 + 2 * (w & 3) + half;
                    const float x = vp_value(key_at(w, half));
                    const int code = coder((x - pv.z[c]) * pv.rinv[c]);
                    if (x < pv.lo[c] || x > pv.hi[c]) outl |= 1u << (w + 16 * half);
                    out |= (uint64_t)(uint32_t)code << (2 * BITS * (2 * (w & 3) + half) + BITS * (w >> 2));
                }
            }
        }
        // ranks: channel order is the head's lower channels, then its upper ones
        const uint32_t n_low = (uint32_t)__popc(outl & 0x000F000Fu), n_up = (uint32_t)__popc(outl & 0x00F000F0u);
        uint32_t in_head = n_low | n_up << 16;                             // up to this lane, within the head
        {
            const uint32_t a = vp_dpp<0x111>(0u, in_head);
            in_head += l8 >= 1 ? a : 0u;
            const uint32_t b = vp_dpp<0x112>(0u, in_head);
            in_head += l8 >= 2 ? b : 0u;
            const uint32_t c = vp_dpp<0x114>(0u, in_head);
            in_head += l8 >= 4 ? c : 0u;
        }
        uint32_t head_low = n_low;                                         // of the head
        head_low += vp_dpp<0xB1>(0u, head_low);
        head_low += vp_dpp<0x4E>(0u, head_low);
        head_low += vp_dpp<0x141>(0u, head_low);
        const uint32_t upto = vp_scan(n_low + n_up);
        uint32_t *sums = wave_sum[t & 1];
        if (lane == 63) sums[wave] = upto;
        __syncthreads();
        uint32_t total = 0, rank_low = upto - ((in_head & 0xFFFFu) + (in_head >> 16));
        {
            static_assert(KVQ_BULK_MAX_WAVES == 8, "two loads");
            const uint4 a = *(const uint4 *)sums, b = *(const uint4 *)(sums + 4);
            const uint32_t n[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                rank_low += w < wave ? n[w] : 0u;
                total += n[w];
            }
        }
        const uint32_t rank_up = rank_low + head_low + (in_head >> 16) - n_up;
        rank_low += (in_head & 0xFFFFu) - n_low;
        for (uint32_t left = outl; __ballot(left != 0u) != 0ull;) {
            if (left == 0u) continue;
            const int b = __ffs((int)left) - 1, w = b & 7, half = b >> 4, up = w >> 2;
            left &= left - 1u;
            const int f = 2 * (w & 3) + half, c = c0 + 64 * up + f;
            const float x = vp_value(key_at(w, half));
            const uint16_t sb = ((const uint16_t *)&bulk_s[(2 + up) * NT + tid])[f], zb = ((const uint16_t *)&bulk_s[(4 + up) * NT + tid])[f];
            int code = (int)(uint32_t)(out >> (2 * BITS * f + BITS * up)) & (NE - 1);
            // Beyond KVQ_CODE_RANGE the thresholds do not give the code, and the outlier thresholds usually lie within it.  (First a test that
            // needs no reciprocal: fp32 steps shift it by less than one in 2^21, so 126 scales are surely within 127.)
            const float diff = x - kvq_h2f(zb);
            if (!(__builtin_fabsf(diff) <= 126.0f * kvq_h2f(sb))) {
                static_assert(KVQ_CODE_RANGE == 127.0f, "see above");
                const float xn = diff * pv.rinv[c];
                if (!(__builtin_fabsf(xn) <= KVQ_CODE_RANGE)) {
                    float unused;
                    code = kvq_nearest<NE>(pv.hdr->lut_k, xn, unused);
                    const int at = 2 * BITS * f + BITS * up;
                    out = (out & ~((uint64_t)(NE - 1) << at)) | (uint64_t)(uint32_t)code << at;
                }
            }
            const uint32_t lower = (((1u << w) - 1u) & (up ? 0xF0u : 0x0Fu)) * 0x00010001u | (half ? 1u << w : 0u);
            const uint64_t pos = base + (up ? rank_up : rank_low) + (uint32_t)__popc(outl & lower);
            if (pos < (uint64_t)cap_nnz)
                ksp.put(pos, (uint16_t)c, kvq_f2h_rn(x - __builtin_fmaf(kvq_h2f(sb), lut_s[code], kvq_h2f(zb))));
            else overflow = true;
        }
        base += total;
        const int64_t n = n0 + t;
        if (tid == 0) {
            k_ptr[n + 1] = (uint32_t)(base > (uint64_t)cap_nnz ? (uint64_t)cap_nnz : base);
            overflow = overflow || base > (uint64_t)cap_nnz;
        }
        uint8_t *chunk = k_codes + kvq_k_piece0(BITS, cap, n, h);
        const uint32_t lo = (uint32_t)out, up = (uint32_t)(out >> 32);
        if constexpr (BITS == 4) {
            *(uint2 *)(chunk + (l8 >> 1) * 1024 + (l8 & 1) * 8) = uint2{lo, up};
        } else if constexpr (BITS == 2) {
            *(uint32_t *)(chunk + (l8 >> 2) * 1024 + (l8 & 3) * 4) = lo;
        } else {
            // 48 bits a lane: an even lane and its neighbour have three dwords
            const uint32_t from_odd = vp_dpp<0xB1>(0u, lo);
            const int d = 3 * (l8 >> 1) + ((l8 & 1) ? 2 : 0);
            *(uint32_t *)(chunk + (d >> 2) * 1024 + (d & 3) * 4) = (l8 & 1) ? (uint32_t)(out >> 16) : lo;
            if (!(l8 & 1)) *(uint32_t *)(chunk + ((d + 1) >> 2) * 1024 + ((d + 1) & 3) * 4) = (up & 0xFFFFu) | from_odd << 16;
        }
    }
    if (overflow) atomicExch(d_status, (int32_t)KVQ_ERR_NNZ_OVERFLOW);
}

}  // namespace

void kvq_k_bulk_launch(const kvq_cache *c, const uint16_t *d_k_new, int T, const uint32_t *counts, hipStream_t s)
{
    const int D = c->n_kv_heads * KVQ_HEAD_DIM;
    const auto launch = [&](auto bits, const auto ksp) {
        const int run = kvq_k_bulk_run(decltype(bits)::value, D, T);
        kvq_k_bulk<decltype(bits)::value><<<kvq_xcd_grid((T + run - 1) / run), D / 16, 6 * D, s>>>(
            c->params, D, c->cap_tokens, c->n_tokens_k, T, run, d_k_new, counts, c->k_codes, c->k_ptr, ksp, c->cap_nnz_k, c->d_status);
    };
    const auto by_bits = [&](const auto ksp) {
        if (c->bits == 2) launch(std::integral_constant<int, 2>{}, ksp);
        else if (c->bits == 3) launch(std::integral_constant<int, 3>{}, ksp);
        else launch(std::integral_constant<int, 4>{}, ksp);
    };
    if (c->nnz_block_shift) by_bits(kvq_blocked_k(c));
    else by_bits(kvq_flat_k(c));
}
