// fp16 numbers as signed 16-bit keys in the order of the values, two to a register (kvq_v_pair.hip, kvq_k_bulk.hip, kvq_lut_load).
#pragma once
#include "kvq_common.hpp"

// Bits 3 and 4 of kvq_cache.loaded, set by kvq_lut_load too: the Keys' (the Values') codes cannot be counted with thresholds (KVQ_CODE_RANGE).
#define KVQ_LOADED_SEARCH_K 8
#define KVQ_LOADED_SEARCH_V 16

namespace {

typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ s16x2 vp_keys(uint32_t two)                     // and back again
{
    const s16x2 x = __builtin_bit_cast(s16x2, two);
    const uint32_t sign = __builtin_bit_cast(uint32_t, x >> (short)15);
    return __builtin_bit_cast(s16x2, two ^ (sign & 0x7FFF7FFFu));
}
__device__ __forceinline__ float vp_value(int key)
{
    return kvq_h2f((uint16_t)(key ^ ((key >> 15) & 0x7FFF)));
}
__device__ __forceinline__ int vp_key(float x)                              // of x rounded to fp16
{
    const int b = (int16_t)kvq_f2h_rn(x);
    return b ^ ((b >> 15) & 0x7FFF);
}
__device__ __forceinline__ uint32_t vp_word(s16x2 v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ s16x2 vp_both(int k) { return s16x2{(short)k, (short)k}; }
__device__ __forceinline__ s16x2 vp_pair(uint32_t w) { return __builtin_bit_cast(s16x2, w); }
// All ones where a < b.  (The empty asm: the compiler would turn masks back into comparisons of either half, and a selection by mask into five
// instructions.)
__device__ __forceinline__ uint32_t vp_less(s16x2 a, s16x2 b)
{
    uint32_t m = vp_word(__builtin_elementwise_sub_sat(a, b) >> (short)15);
    asm("" : "+v"(m));
    return m;
}
__device__ __forceinline__ uint32_t vp_select(uint32_t mask, uint32_t a, uint32_t b) { return (mask & a) | (~mask & b); }

template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ uint32_t vp_dpp(uint32_t old, uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROWS, 0xf, false);
}
// Sums over the lanes up to and including this one.
__device__ __forceinline__ uint32_t vp_scan(uint32_t v)
{
    v += vp_dpp<0x111>(0u, v);
    v += vp_dpp<0x112>(0u, v);
    v += vp_dpp<0x114>(0u, v);
    v += vp_dpp<0x118>(0u, v);
    v += vp_dpp<0x142, 0xa>(0u, v);            // lane 15 of rows 0 and 2 into rows 1 and 3
    v += vp_dpp<0x143, 0xc>(0u, v);            // lane 31 into rows 2 and 3
    return v;
}

// The part of the parameter block (behind kvq_params_bytes_D(D) bytes) for the bulk Key append.
struct KvqKeyParams {
    const int16_t *thr;          // [15][D] the smallest key that reaches a code threshold
    const int16_t *first, *last; // [D] the first and the last key that is no outlier and within KVQ_CODE_RANGE
    const uint8_t *narrow;       // [D / 8] a bit per channel: its range ends at KVQ_CODE_RANGE, not at an outlier threshold
};
__host__ __device__ inline int64_t kvq_key_params_bytes(int D) { return (int64_t)D * 17 * 2 + D / 8; }
__host__ __device__ inline KvqKeyParams kvq_key_params(const void *block, int D)
{
    KvqKeyParams v;
    v.thr = (const int16_t *)((const char *)block + kvq_params_bytes_D(D));
    v.first = v.thr + (int64_t)15 * D;
    v.last = v.first + D;
    v.narrow = (const uint8_t *)(v.last + D);
    return v;
}

// The smallest key whose normalised value (x - z) * rinv reaches `thr` (31744: no finite one does), for finite z and rinv > 0.  It is next to
// where the inverse of the normalisation points; thresholds past the largest number and scales of few bits are searched for.
__device__ __forceinline__ int vp_first_key(float thr, float s, float z, float rinv)
{
    auto reaches = [&](int key) { return (vp_value(key) - z) * rinv >= thr; };
    const int guess = vp_key(__builtin_fmaf(thr, s, z));
    int below = 0;
    bool first = false, last = false;
#pragma unroll
    for (int i = -2; i <= 2; ++i) {
        const bool r = reaches(guess + i);
        below += r ? 0 : 1;
        if (i == -2) first = r;
        if (i == 2) last = r;
    }
    int k = guess - 2 + below;
    if (first || !last) {
        int a = -31744, b = 31744;                       // keys of finite numbers, and none
        while (a < b) {
            const int mid = (a + b) >> 1;
            if (reaches(mid)) b = mid;
            else a = mid + 1;
        }
        k = a;
    }
    return k;
}

}  // namespace
