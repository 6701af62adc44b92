// Pieces of the radix selections on fp16 values, shared by the per-token Value outliers of the appends
// and the per-channel Key thresholds of the offline calibration.
#pragma once
#include "kvq_common.hpp"

namespace {

// Order-preserving 16-bit key of an fp16 bit pattern (-0 is treated as +0).
__device__ inline uint32_t order_key(uint16_t h)
{
    if (h == 0x8000u) h = 0;
    return (h & 0x8000u) ? (uint32_t)(uint16_t)~h : (uint32_t)(h | 0x8000u);
}

// The value of a key.
__device__ inline float key_value(uint32_t key)
{
    return kvq_h2f((uint16_t)((key & 0x8000u) ? (key & 0x7FFFu) : (~key & 0xFFFFu)));
}

// In a histogram of 256 bins (lane l reads bins 4l..4l+3), the bin in which the K-th element counted
// from the top (FROM_TOP) or from the bottom lies, the number of elements beyond that bin on that side,
// and the bin's own count.  Wavefront-uniform results.  1 <= K <= number of elements.
template <bool FROM_TOP>
__device__ __forceinline__ void wave_find_bin(const uint32_t *h256, uint32_t K, int lane, uint32_t &bin,
                                              uint32_t &beyond, uint32_t &in_bin)
{
    const uint4 v = *(const uint4 *)(h256 + 4 * lane);
    const uint32_t hh[4] = {v.x, v.y, v.z, v.w};
    const uint32_t s = v.x + v.y + v.z + v.w;
    uint32_t S = s;                                // sum over this lane and the lanes on the side counted from
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = FROM_TOP ? __shfl_down(S, o) : __shfl_up(S, o);
        if (FROM_TOP ? (lane + o < 64) : (lane >= o)) S += t;
    }
    uint32_t a = S - s;                            // elements in the bins of the lanes beyond this one
    int found = -1;
    uint32_t fa = 0, fh = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int q = FROM_TOP ? 3 - i : i;
        if (found < 0 && a < K && a + hh[q] >= K) { found = q; fa = a; fh = hh[q]; }
        a += hh[q];
    }
    const int src = __ffsll((unsigned long long)__ballot(found >= 0)) - 1;      // exactly one lane finds it
    bin = (uint32_t)__shfl(4 * lane + found, src);
    beyond = __shfl(fa, src);
    in_bin = __shfl(fh, src);
}

}  // namespace
