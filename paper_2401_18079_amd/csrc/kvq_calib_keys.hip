// Offline per-channel calibration of the Keys (paper Sec. 3.6 and the appendix on offline calibration):
// per channel the k smallest and the k largest of the T calibration values are its outliers; thresholds
// are the k-th smallest / largest value, and the values strictly inside give the zero-point (mid-range)
// and scale (half-range).  With the channel's values sorted these are four order statistics: the k-th
// and the (k+1)-th from either end.
//
// Design (gfx950).  The matrix is [T][D], a channel a column of it, and no scratch memory comes with the
// call, so a workgroup owns a group of neighbouring channels from the first row to the last: a load
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

// LPR lanes of V channels each: a workgroup owns C = V * LPR channels.
template <int V, int LPR>
__global__ __launch_bounds__(CK_NT) __attribute__((amdgpu_waves_per_eu(LPR == 2 ? 4 : 8)))
void kvq_calib_channels(const uint16_t *__restrict__ k_cal, int T, int D, int k, int groups,
                        uint16_t *__restrict__ s_out, uint16_t *__restrict__ z_out, uint16_t *__restrict__ lo_out,
                        uint16_t *__restrict__ hi_out)
{
    constexpr int C = V * LPR;
    static_assert(C <= CK_NT / 64, "a wavefront per channel finds its bins");
    // [C][4][256]: low-byte counts; the high-byte counts of sweep one are the same memory's first quarter
    __shared__ __attribute__((aligned(16))) uint32_t cnt[C * 4 * 256];
    __shared__ uint32_t bound[C];          // (first counted upper bin) << 8 | (last counted lower bin)
    __shared__ uint32_t target[C];         // bins of the order statistics: top k, top k+1, bottom k, bottom k+1
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // consecutive groups on one XCD: block b of 8 n runs on XCD b mod 8
    int g = (int)blockIdx.x;
    if ((groups & 7) == 0) g = (g & 7) * (groups >> 3) + (g >> 3);
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
    if (lane == 0) {
        const int c = g * C + wave;
        uint16_t hb, lob, unused;
        const float a = ck_value(key[3], unused), b = ck_value(key[1], unused);
        ck_value(key[0], hb);
        ck_value(key[2], lob);
        const uint16_t zc = kvq_f2h_rn((b + a) * 0.5f);
        uint16_t sc = kvq_f2h_rn((b - a) * 0.5f);
        if (!(kvq_h2f(sc) > 0.0f)) sc = 0x3C00u;                      // 1.0
        s_out[c] = sc;
        z_out[c] = zc;
        lo_out[c] = (k > 0) ? lob : (uint16_t)0xFBFFu;                // -65504
        hi_out[c] = (k > 0) ? hb : (uint16_t)0x7BFFu;                 // +65504
    }
}

}  // namespace

extern "C" kvq_status kvq_calibrate_key_channels(const uint16_t *d_k_cal, int32_t T, int32_t D, float outlier_fraction,
                                                 uint16_t *d_s, uint16_t *d_z, uint16_t *d_lo, uint16_t *d_hi,
                                                 void *stream)
{
    if (!d_k_cal || !d_s || !d_z || !d_lo || !d_hi || ((uintptr_t)d_k_cal & 1)) return KVQ_ERR_INVALID_ARG;
    if (T < 1 || D < 1 || !(outlier_fraction >= 0.0f) || !(outlier_fraction < 1.0f)) return KVQ_ERR_INVALID_ARG;
    if (T > 32768) return KVQ_ERR_UNSUPPORTED;
    const int k = (int)floorf(outlier_fraction * 0.5f * (float)T + 0.5f);
    if (2 * k >= T) return KVQ_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    // The widest group that divides D, whose loads are aligned, and that still gives a workgroup per compute
    // unit (a group is swept by one workgroup from end to end).  Measured on 32768 x 4096: groups of 32
    // channels (64-byte pieces, half the compute units) 272 us, of 16 182 us, of 8 (16-byte pieces) 248 us.
    const int64_t cus = kvq_cu_count();
    auto fits = [&](int v, int c) {
        return D % c == 0 && ((uintptr_t)d_k_cal & (2 * v - 1)) == 0 && (c == 1 || (int64_t)D / c >= cus);
    };
#define LAUNCH_CK(V, LPR)                                                                                          \
    kvq_calib_channels<V, LPR><<<D / ((V) * (LPR)), CK_NT, 0, s>>>(d_k_cal, T, D, k, D / ((V) * (LPR)), d_s, d_z,   \
                                                                   d_lo, d_hi)
    if (fits(8, 16)) LAUNCH_CK(8, 2);
    else if (fits(8, 8)) LAUNCH_CK(8, 1);
    else if (fits(4, 4)) LAUNCH_CK(4, 1);
    else if (fits(2, 2)) LAUNCH_CK(2, 1);
    else LAUNCH_CK(1, 1);
#undef LAUNCH_CK
    KVQ_HIP_CHECK(hipGetLastError());
    return KVQ_OK;
}
