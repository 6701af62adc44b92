// Offline derivation of the non-uniform datatype (paper Sec. 3.3, Eq. (1), with the s_i^2 weighting of
// the appendix on per-channel scaling): the 2^b signposts that minimise
//     sum_i w_i (x_i - Q(x_i))^2,   w_i = F_ii s_i^2,   x = normalised calibration activations,
// found with Lloyd's k-means iteration in one dimension.
//
// Design (gfx950).  An iteration streams the n values and weights once (8 bytes per element: HBM-bound for
// large n) and needs, per signpost, the sums of w and of w*x over the elements nearest to it.  The index of
// the nearest signpost is data dependent, so the running sums cannot live in registers; every lane owns a
// private column of fp64 accumulators in LDS ([signpost][lane]: no atomics, no bank conflicts).  The index
// comes from a search over all signposts or, for 16 of them and many elements, from a look-up: the update that moves
// the signposts also finds the exact decision thresholds between them (KVQ_CODE_RANGE), a workgroup spreads these
// over 1024 cells of [-1, 1], and an element reads its cell's index and compares with the one threshold in it.  Where
// two thresholds fall into one cell, or the signposts are not monotone to count on, and for values far outside, the
// search decides there too.  Workgroups write their sums to a workspace, and a one-workgroup kernel adds them in a
// fixed order and moves the signposts, which stay on the device between iterations.  fp32 distances with ties to the
// smaller index decide the assignment; sums are fp64 (w*x of two fp32 numbers is exact in fp64).
// Measured per iteration on 33.6 M elements, 16 signposts: 78 us and 10 us for the update with the search (four
// instructions per signpost), loads not ahead of it, and a four-wavefront update; 46 us and 8 us now.  On 65536
// elements, where the search is taken: 5.0 and 2.3 us.
#include <algorithm>
#include <type_traits>
#include "kvq_common.hpp"

namespace {

constexpr int CAL_NT = 256;
constexpr int CAL_MAX_WGS = 2048;
constexpr int64_t CAL_LOOK_UP_MIN = 6 << 20;      // elements from which 16 signposts are found by look-up
constexpr int CAL_PARTS = 64;            // partial sums per signpost in the update kernel

template <int K>
__device__ __forceinline__ int cal_nearest(const float (&c)[K], float x)
{
    int best = 0;
    float bestd = __builtin_fabsf(x - c[0]);
#pragma unroll
    for (int j = 1; j < K; ++j) {
        const float d = __builtin_fabsf(x - c[j]);
        if (d < bestd) { bestd = d; best = j; }
    }
    return best;
}

constexpr int CAL_CELLS = 1024;
__device__ __forceinline__ uint32_t cal_cell(float x)             // monotone in x
{
    const float c = __builtin_fmaf(x, CAL_CELLS / 2, CAL_CELLS / 2);
    return (uint32_t)__builtin_amdgcn_fmed3f(c, 0.0f, (float)(CAL_CELLS - 1));
}

// partial[workgroup][K][2] = (sum of w, sum of w*x) over the workgroup's elements nearest to signpost j.
// cent: K signposts, and from cent[16] on their K - 1 thresholds (thr[0] NaN: not to be counted on).
// 33.6 M elements, 16 signposts: 78 -> 46 us (268 MB: 5.8 TB/s); bound by HBM.
// LOOK_UP = false: every element takes the search (see run_calibration).
template <int K, bool LOOK_UP>
__global__ __launch_bounds__(CAL_NT) void kvq_calib_assign(const float *__restrict__ x, const float *__restrict__ w,
                                                           int64_t n, const float *__restrict__ cent,
                                                           double *__restrict__ partial)
{
    __shared__ double2 acc[K][CAL_NT];
    __shared__ float2 cells[LOOK_UP ? CAL_CELLS : 1];        // (threshold inside the cell or +inf, index below it)
    __shared__ int crowded;
    const int tid = threadIdx.x;
    const float *thr = cent + 16;
    for (int j = 0; j < K; ++j) acc[j][tid] = double2{0.0, 0.0};
    if (LOOK_UP) {
        if (tid == 0) crowded = !(thr[0] == thr[0]);
        __syncthreads();
    }
    for (int c = tid; c < (LOOK_UP ? CAL_CELLS : 0); c += CAL_NT) {
        int below = 0, inside = 0;
        float t = INFINITY;
#pragma unroll
        for (int j = 0; j < K - 1; ++j) {
            const float tj = thr[j];
            const uint32_t cj = cal_cell(tj);
            below += cj < (uint32_t)c ? 1 : 0;
            if (cj == (uint32_t)c) { t = tj; ++inside; }
        }
        cells[c] = float2{t, __builtin_bit_cast(float, below)};
        if (inside > 1) crowded = 1;
    }
    if (LOOK_UP) __syncthreads();
    const bool look_up = LOOK_UP && !crowded;
    // groups of four consecutive elements per lane (16-byte loads), grid-stride over the groups; two groups
    // ahead are in flight (two workgroups per compute unit is all that the accumulators of 16 signposts leave)
    const int64_t n4 = n >> 2, stride = (int64_t)gridDim.x * CAL_NT;
    const float4 *x4 = (const float4 *)x, *w4 = (const float4 *)w;
    auto add = [&](int j, float xe, float we) {
        const double wd = (double)we;
        double2 a = acc[j][tid];
        a.x += wd;
        a.y += wd * (double)xe;
        acc[j][tid] = a;
    };
    auto search = [&](float xe) {
        float c[K];
#pragma unroll
        for (int j = 0; j < K; ++j) c[j] = cent[j];
        return cal_nearest<K>(c, xe);
    };
    auto take = [&](const float4 &xv, const float4 &wv) {
        const float xs[4] = {xv.x, xv.y, xv.z, xv.w}, ws[4] = {wv.x, wv.y, wv.z, wv.w};
        int j[4];
        bool far = !look_up;
#pragma unroll
        for (int e = 0; e < 4; ++e) far = far || !(__builtin_fabsf(xs[e]) <= KVQ_CODE_RANGE);
        if (__ballot(far) != 0ull) {
#pragma unroll
            for (int e = 0; e < 4; ++e) j[e] = search(xs[e]);
        } else {
            float2 c[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) c[e] = cells[cal_cell(xs[e])];
#pragma unroll
            for (int e = 0; e < 4; ++e) j[e] = __builtin_bit_cast(int, c[e].y) + (xs[e] >= c[e].x ? 1 : 0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) add(j[e], xs[e], ws[e]);
    };
    const int64_t g0 = (int64_t)blockIdx.x * CAL_NT + tid, last = n4 - 1;
    float4 xa = {}, wa = {}, xb = {}, wb = {};
    if (n4 > 0) {                              // (indexes past the end re-read the last group)
        xa = x4[g0 < last ? g0 : last];
        wa = w4[g0 < last ? g0 : last];
        xb = x4[g0 + stride < last ? g0 + stride : last];
        wb = w4[g0 + stride < last ? g0 + stride : last];
    }
    for (int64_t g = g0; g < n4; g += 2 * stride) {
        const int64_t ga = g + 2 * stride < last ? g + 2 * stride : last, gb = g + 3 * stride < last ? g + 3 * stride : last;
        const float4 xn = x4[ga], wn = w4[ga];
        take(xa, wa);
        xa = xn; wa = wn;
        const float4 xm = x4[gb], wm = w4[gb];
        if (g + stride < n4) take(xb, wb);
        xb = xm; wb = wm;
    }
    // the last n % 4 elements
    if (blockIdx.x == 0 && tid < (int)(n & 3)) {
        const int64_t i = (n4 << 2) + tid;
        add(search(x[i]), x[i], w[i]);
    }
    __syncthreads();
    // columns are added up in a fixed order: PARTS threads per row of sums, each every PARTS-th column (next to each
    // other in the banks), then their sums
    constexpr int PARTS = CAL_NT / (2 * K);
    const double *sums = (const double *)&acc[0][0];
    const int row = tid / PARTS, part = tid % PARTS;        // row: 2 j + (0: w, 1: w x)
    double s = 0.0;
    for (int l = part; l < CAL_NT; l += PARTS) s += sums[((row >> 1) * CAL_NT + l) * 2 + (row & 1)];
    __syncthreads();
    double *parts = (double *)&acc[0][0];
    parts[tid] = s;
    __syncthreads();
    if (tid < 2 * K) {
        double t = 0.0;
        for (int p = 0; p < PARTS; ++p) t += parts[tid * PARTS + p];
        partial[(int64_t)blockIdx.x * K * 2 + tid] = t;
    }
}

// cent[j] = fp32(sum w x / sum w) over all workgroups' partial sums, in a fixed order; a signpost
// whose elements weigh nothing stays where it is.  Then the thresholds between the signposts.  n_wgs = 0: only
// the thresholds.
template <int K, bool LOOK_UP>
__global__ __launch_bounds__(CAL_PARTS * 16) void kvq_calib_update(const double *__restrict__ partial, int n_wgs,
                                                                   float *__restrict__ cent)
{
    __shared__ double2 sums[CAL_PARTS][16];
    __shared__ float c[K];
    const int j = threadIdx.x & 15, part = threadIdx.x >> 4;
    double2 a = {0.0, 0.0};
    if (j < K) {
        for (int g0 = part; g0 < n_wgs; g0 += 8 * CAL_PARTS) {          // eight loads in flight per thread
            double2 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int g = g0 + u * CAL_PARTS;
                v[u] = g < n_wgs ? *(const double2 *)(partial + ((int64_t)g * K + j) * 2) : double2{0.0, 0.0};
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) { a.x += v[u].x; a.y += v[u].y; }
        }
    }
    sums[part][j] = a;
    __syncthreads();
    if (part == 0 && j < K) {
        double ta = 0.0, tb = 0.0;
        for (int p = 0; p < (n_wgs < CAL_PARTS ? n_wgs : CAL_PARTS); ++p) { ta += sums[p][j].x; tb += sums[p][j].y; }
        c[j] = ta > 0.0 ? (float)(tb / ta) : cent[j];
        cent[j] = c[j];
    }
    if (!LOOK_UP) return;
    __syncthreads();
    if (threadIdx.x >= K - 1) return;
    // thr[j]: the smallest fp32 x in the range that lies nearer to the next signpost above c[j] (strictly: a tie
    // goes to the smaller index), by bisection over the ordered fp32 numbers
    bool counted = true;
    for (int i = 0; i < K; ++i) {
        counted = counted && __builtin_fabsf(c[i]) <= 1.0f;
        if (i > 0) counted = counted && (c[i] == c[i - 1] || c[i] - c[i - 1] >= KVQ_CODE_MIN_GAP);
    }
    const int t = threadIdx.x;
    const float v = c[t];
    float up = INFINITY;
    for (int i = K - 1; i > t; --i) up = c[i] > v ? c[i] : up;
    float out = INFINITY;
    if (up <= 1.0f) {
        auto val = [](int64_t k) { return __builtin_bit_cast(float, (int32_t)(k >= 0 ? k : (int64_t)INT32_MIN - k)); };
        const int64_t top = (int64_t)__builtin_bit_cast(int32_t, KVQ_CODE_RANGE);
        int64_t lo = -top, hi = top;            // (the range's ends lie nearer to the lower and to the upper signpost)
        while (lo < hi) {
            const int64_t mid = lo + ((hi - lo) >> 1);
            const float m = val(mid);
            if (__builtin_fabsf(m - up) < __builtin_fabsf(m - v)) hi = mid;
            else lo = mid + 1;
        }
        out = val(lo);
    }
    cent[16 + t] = counted ? out : __builtin_nanf("");
}

template <int K>
kvq_status run_calibration(const float *x, const float *w, int64_t n, int iters, float *cent, double *partial,
                           hipStream_t s)
{
    // enough workgroups to fill the chip (LDS allows 6 / 3 / 2 per compute unit for 4 / 8 / 16 signposts),
    // no more than there are groups of 1024 elements, within the workspace's slots
    int64_t wgs = (n / 4 + CAL_NT - 1) / CAL_NT;
    const int64_t fill = (int64_t)kvq_cu_count() * (K == 16 ? 2 : K == 8 ? 3 : 6);
    if (wgs > fill) wgs = fill;
    if (wgs > CAL_MAX_WGS) wgs = CAL_MAX_WGS;
    if (wgs < 1) wgs = 1;
    auto run = [&](auto look_up) {
        constexpr bool LU = decltype(look_up)::value;
        if (LU && iters > 0) kvq_calib_update<K, LU><<<1, CAL_PARTS * 16, 0, s>>>(partial, 0, cent);      // the first thresholds
        for (int it = 0; it < iters; ++it) {
            kvq_calib_assign<K, LU><<<(unsigned)wgs, CAL_NT, 0, s>>>(x, w, n, cent, partial);
            kvq_calib_update<K, LU><<<1, CAL_PARTS * 16, 0, s>>>(partial, (int)wgs, cent);
        }
    };
    // The look-up saves the search's four instructions per signpost and element and costs 3 us (4 signposts) to 5 us
    // (16) per iteration for the thresholds and the workgroups' cells.  Whole calls of 20 iterations, us, look-up
    // against search: 16 signposts, 100000 elements 310 / 210, 1 M 385 / 275, 4.2 M 432 / 407, 8.4 M 558 / 586, 16.8 M 729 / 938;
    // 8 signposts, 100000 elements 278 / 202, 16.8 M 763 / 699; 4 signposts, 16.8 M 780 / 712.
    if constexpr (K == 16) {
        if (n >= CAL_LOOK_UP_MIN) run(std::true_type{});
        else run(std::false_type{});
    } else {
        run(std::false_type{});
    }
    KVQ_HIP_CHECK(hipGetLastError());
    return KVQ_OK;
}

}  // namespace

extern "C" int64_t kvq_calibrate_workspace_bytes(void)
{
    return (int64_t)CAL_MAX_WGS * 16 * 2 * (int64_t)sizeof(double) + 256;
}

extern "C" kvq_status kvq_calibrate_nuq(const float *d_x_norm, const float *d_w, int64_t n, int32_t bits,
                                        int32_t iters, float *h_signposts, void *d_workspace,
                                        int64_t workspace_bytes, void *stream)
{
    if (!d_x_norm || !d_w || !h_signposts || !d_workspace) return KVQ_ERR_INVALID_ARG;
    if (((uintptr_t)d_x_norm & 15) || ((uintptr_t)d_w & 15) || ((uintptr_t)d_workspace & 255)) return KVQ_ERR_INVALID_ARG;
    if (n < 1 || iters < 0) return KVQ_ERR_INVALID_ARG;
    if (bits < 2 || bits > 4) return KVQ_ERR_UNSUPPORTED;
    if (workspace_bytes < kvq_calibrate_workspace_bytes()) return KVQ_ERR_CAPACITY;
    hipStream_t s = (hipStream_t)stream;
    const int K = 1 << bits;
    float *cent = (float *)d_workspace;                       // 16 signposts, 15 thresholds, then the partial sums
    double *partial = (double *)((char *)d_workspace + 256);
    KVQ_HIP_CHECK(hipMemcpyAsync(cent, h_signposts, (size_t)K * sizeof(float), hipMemcpyHostToDevice, s));
    kvq_status st = (bits == 2)   ? run_calibration<4>(d_x_norm, d_w, n, iters, cent, partial, s)
                    : (bits == 3) ? run_calibration<8>(d_x_norm, d_w, n, iters, cent, partial, s)
                                  : run_calibration<16>(d_x_norm, d_w, n, iters, cent, partial, s);
    if (st != KVQ_OK) return st;
    KVQ_HIP_CHECK(hipMemcpyAsync(h_signposts, cent, (size_t)K * sizeof(float), hipMemcpyDeviceToHost, s));
    KVQ_HIP_CHECK(hipStreamSynchronize(s));
    std::sort(h_signposts, h_signposts + K);
    return KVQ_OK;
}
