// Offline derivation of the non-uniform datatype (paper Sec. 3.3, Eq. (1), with the s_i^2 weighting of
// the appendix on per-channel scaling): the 2^b signposts that minimise
//     sum_i w_i (x_i - Q(x_i))^2,   w_i = F_ii s_i^2,   x = normalised calibration activations,
// found with Lloyd's k-means iteration in one dimension.
//
// Design (gfx950).  An iteration streams the n values and weights once (8 bytes per element: HBM-bound for
// large n) and needs, per signpost, the sums of w and of w*x over the elements nearest to it.  The index of
// the nearest signpost is data dependent, so the running sums cannot live in registers; every lane owns a
// private column of fp64 accumulators in LDS ([signpost][lane]: no atomics, no bank conflicts).  The index
// comes from a search over all signposts or, for 16 of them and many elements, from a look-up: a workgroup finds the exact
// decision thresholds between the signposts (KVQ_CODE_RANGE) and spreads them over 1024 cells of [-1, 1]; an element reads its
// cell's index and compares with the one threshold in it.  Where two thresholds fall into one cell, or the signposts are not
// monotone to count on, and for values far outside, the search decides there too.  Workgroups write their sums to a workspace, and
// every workgroup of the next iteration's launch adds them up for itself, in a fixed order, before it starts: an iteration is one
// launch.  fp32 distances with ties to the smaller index decide the assignment; sums are fp64 (w*x of two fp32 numbers is exact
// in fp64).
// 20 iterations, us, with a launch of one workgroup between two iterations that moved the signposts, and now: 16 signposts,
// 33.6 M elements 1093 / 991, 4 M 379 / 292, 1 M 243 / 203, 100000 195 / 178; 4 signposts, 33.6 M 1018 / 887, 1 M 211 / 175.
// Bound: HBM (an iteration over 33.6 M elements, 268 MB, takes 49 us, 5.5 TB/s) behind 9 us per iteration of launch, sums, thresholds and
// cells.  Sweeps alternately from either end, for the last-level cache: no change; four groups ahead instead of two: 2 % slower.
#include <algorithm>
#include <type_traits>
#include "kvq_common.hpp"

namespace {

constexpr int CAL_NT = 512;
constexpr int CAL_MAX_WGS = 1024;
constexpr int64_t CAL_LOOK_UP_MIN = 3 << 20;      // elements from which 16 signposts are found by look-up

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

// What an iteration leaves for the next one, twice: an iteration reads one and writes the other.
struct CalState {
    float *cent;              // 16 signposts
    double *partial;          // [workgroup][K][2] = (sum of w, sum of w*x) over its elements nearest to signpost j
};

// The signposts that the sums `from` stand for: c[j] = fp32(sum w x / sum w) over all workgroups, added in a fixed order;
// a signpost whose elements weigh nothing stays where it is.  With n_wgs = 0 they are from.cent itself.  Every workgroup
// of the next launch does this for itself (the sums are 64 KB, and come from its L2).  `scratch`: NT / 64 * K double2.
template <int K>
__device__ __forceinline__ void cal_move(const CalState &from, int n_wgs, double2 *scratch, float *c)
{
    const int tid = threadIdx.x, j = tid % K, part = tid / K;
    constexpr int PARTS = CAL_NT / K;
    double2 a = {0.0, 0.0};
    for (int g0 = part; g0 < n_wgs; g0 += 8 * PARTS) {                  // eight loads in flight per thread
        double2 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int g = g0 + u * PARTS;
            v[u] = *(const double2 *)(from.partial + ((int64_t)(g < n_wgs ? g : g0) * K + j) * 2);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (g0 + u * PARTS < n_wgs) { a.x += v[u].x; a.y += v[u].y; }
        }
    }
#pragma unroll
    for (int o = K; o < 64; o <<= 1) {
        a.x += __shfl_xor(a.x, o);
        a.y += __shfl_xor(a.y, o);
    }
    if ((tid & 63) < K) scratch[(tid >> 6) * K + j] = a;
    __syncthreads();
    if (tid < K) {
        double2 t = {0.0, 0.0};
#pragma unroll
        for (int p = 0; p < CAL_NT / 64; ++p) { t.x += scratch[p * K + tid].x; t.y += scratch[p * K + tid].y; }
        c[tid] = t.x > 0.0 ? (float)(t.y / t.x) : from.cent[tid];
    }
    __syncthreads();
}

// thr[j]: the smallest fp32 x in the range that lies nearer to the next signpost above c[j] (strictly: a tie goes to
// the smaller index), by bisection over the ordered fp32 numbers.  It is within a few roundings of the middle between
// the two, so the bisection starts from a bracket around that (2^-21 of the signposts: a dozen steps at most, unless the middle is near
// zero), and from the whole range where the bracket does not hold the change.  NaN: not to be counted on.
template <int K>
__device__ __forceinline__ float cal_threshold(const float *c, int t)
{
    float s[K];
#pragma unroll
    for (int i = 0; i < K; ++i) s[i] = c[i];
    bool counted = true;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        counted = counted & (__builtin_fabsf(s[i]) <= 1.0f);
        if (i > 0) counted = counted & (s[i] == s[i - 1] | s[i] - s[i - 1] >= KVQ_CODE_MIN_GAP);
    }
    const float v = c[t];
    float up = INFINITY;
#pragma unroll
    for (int i = K - 1; i > 0; --i) up = (i > t & s[i] > v) ? s[i] : up;
    float out = INFINITY;
    if (up <= 1.0f) {
        auto val = [](int64_t k) { return __builtin_bit_cast(float, (int32_t)(k >= 0 ? k : (int64_t)INT32_MIN - k)); };
        auto key = [](float x) {
            const int32_t b = __builtin_bit_cast(int32_t, x);
            return b >= 0 ? (int64_t)b : (int64_t)INT32_MIN - b;
        };
        auto above = [&](int64_t k) { return __builtin_fabsf(val(k) - up) < __builtin_fabsf(val(k) - v); };
        const int64_t top = (int64_t)__builtin_bit_cast(int32_t, KVQ_CODE_RANGE);
        int64_t lo = -top, hi = top;            // (the range's ends lie nearer to the lower and to the upper signpost)
        const float middle = 0.5f * (v + up), reach = (__builtin_fabsf(v) + __builtin_fabsf(up)) * 4.76837158e-7f;
        const int64_t a = key(middle - reach), b = key(middle + reach);
        if (a > lo && b < hi && !above(a) && above(b)) { lo = a; hi = b; }
        while (lo < hi) {
            const int64_t mid = lo + ((hi - lo) >> 1);
            if (above(mid)) hi = mid;
            else lo = mid + 1;
        }
        out = val(lo);
    }
    return counted ? out : __builtin_nanf("");
}

// One iteration: the signposts from the sums of the iteration before, then this one's sums.  The accumulators of 16 signposts are
// 128 KB, so eight wavefronts share a compute unit, and an element's addition is a round trip to LDS: two elements make theirs
// together (four, one after the other, kept the kernel at 5.8 TB/s).
// LOOK_UP = false: every element takes the search (see run_calibration).
template <int K, bool LOOK_UP>
__global__ __launch_bounds__(CAL_NT) void kvq_calib_assign(const float *__restrict__ x, const float *__restrict__ w,
                                                           int64_t n, int n_wgs, const CalState from, const CalState to)
{
    __shared__ __attribute__((aligned(16))) double2 acc[K][CAL_NT];
    __shared__ float2 cells[LOOK_UP ? CAL_CELLS : 1];        // (threshold inside the cell or +inf, index below it)
    __shared__ float cent[K], thr[K];
    __shared__ int crowded;
    const int tid = threadIdx.x;
    // groups of four consecutive elements per lane (16-byte loads), grid-stride over the groups; two groups
    // ahead are in flight (eight wavefronts per compute unit are all that the accumulators of 16 signposts leave)
    const int64_t n4 = n >> 2, stride = (int64_t)gridDim.x * CAL_NT;
    const float4 *x4 = (const float4 *)x, *w4 = (const float4 *)w;
    const int64_t g0 = (int64_t)blockIdx.x * CAL_NT + tid, last = n4 - 1;
    float4 xa = {}, wa = {}, xb = {}, wb = {};
    if (n4 > 0) {                              // (indexes past the end re-read the last group)
        xa = x4[g0 < last ? g0 : last];
        wa = w4[g0 < last ? g0 : last];
        xb = x4[g0 + stride < last ? g0 + stride : last];
        wb = w4[g0 + stride < last ? g0 + stride : last];
    }
    cal_move<K>(from, n_wgs, &acc[0][0], cent);
    if (blockIdx.x == 0 && tid < K) to.cent[tid] = cent[tid];
    if (LOOK_UP) {
        if (tid < K - 1) {
            thr[tid] = cal_threshold<K>(cent, tid);
            if (tid == 0) crowded = !(thr[0] == thr[0]);
        }
        __syncthreads();
        for (int c = tid; c < CAL_CELLS; c += CAL_NT) {
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
    }
    for (int j = 0; j < K; ++j) acc[j][tid] = double2{0.0, 0.0};
    __syncthreads();
    const bool look_up = LOOK_UP && !crowded;
    // two elements at a time: one round trip to the accumulators for both
    auto add2 = [&](const int (&j)[2], const float (&xe)[2], const float (&we)[2]) {
        double2 a = acc[j[0]][tid], b = acc[j[1]][tid];
        const double w0 = (double)we[0], w1 = (double)we[1];
        a.x += w0;
        a.y = __builtin_fma(w0, (double)xe[0], a.y);               // (the product of two fp32 numbers is exact)
        const bool same = j[1] == j[0];
        b.x = (same ? a.x : b.x) + w1;
        b.y = __builtin_fma(w1, (double)xe[1], same ? a.y : b.y);
        acc[j[0]][tid] = a;
        acc[j[1]][tid] = b;
    };
    float sc[LOOK_UP ? 1 : K];
    if (!LOOK_UP) {
#pragma unroll
        for (int j = 0; j < K; ++j) sc[LOOK_UP ? 0 : j] = cent[j];
    }
    auto search = [&](float xe) {
        if constexpr (!LOOK_UP) return cal_nearest<K>(sc, xe);
        float c[K];
#pragma unroll
        for (int j = 0; j < K; ++j) c[j] = cent[j];
        return cal_nearest<K>(c, xe);
    };
    auto take = [&](const float4 &xv, const float4 &wv) {
        const float xs[4] = {xv.x, xv.y, xv.z, xv.w}, ws[4] = {wv.x, wv.y, wv.z, wv.w};
        int j[4];
        bool far = !look_up;
        if (LOOK_UP) {
#pragma unroll
            for (int e = 0; e < 4; ++e) far = far || !(__builtin_fabsf(xs[e]) <= KVQ_CODE_RANGE);
        }
        if (!LOOK_UP || __ballot(far) != 0ull) {
#pragma unroll
            for (int e = 0; e < 4; ++e) j[e] = search(xs[e]);
        } else {
            float2 c[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) c[e] = cells[cal_cell(xs[e])];
#pragma unroll
            for (int e = 0; e < 4; ++e) j[e] = __builtin_bit_cast(int, c[e].y) + (xs[e] >= c[e].x ? 1 : 0);
        }
        add2({j[0], j[1]}, {xs[0], xs[1]}, {ws[0], ws[1]});
        add2({j[2], j[3]}, {xs[2], xs[3]}, {ws[2], ws[3]});
    };
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
        const int j = search(x[i]);
        const double wd = (double)w[i];
        acc[j][tid].x += wd;
        acc[j][tid].y = __builtin_fma(wd, (double)x[i], acc[j][tid].y);
    }
    __syncthreads();
    // columns are added up in a fixed order: PARTS threads per row of sums, each every PARTS-th column (next to each
    // other in the banks), then their sums
    constexpr int PARTS = CAL_NT / (2 * K);
    const double *sums = (const double *)&acc[0][0];
    const int row = tid / PARTS, part = tid % PARTS;        // row: 2 j + (0: w, 1: w x)
    double s = 0.0;
    for (int l = part; l < CAL_NT; l += PARTS) s += sums[((row >> 1) * CAL_NT + l) * 2 + (row & 1)];
#pragma unroll
    for (int o = 1; o < (PARTS < 64 ? PARTS : 64); o <<= 1) s += __shfl_xor(s, o);
    if constexpr (PARTS <= 64) {
        if (part == 0) to.partial[(int64_t)blockIdx.x * K * 2 + row] = s;
    } else {
        static_assert(PARTS <= 64, "a row's partial sums lie in one wavefront");
    }
}

// The signposts after the last iteration, to out.
template <int K>
__global__ __launch_bounds__(CAL_NT) void kvq_calib_finish(int n_wgs, const CalState from, float *__restrict__ out)
{
    __shared__ double2 scratch[CAL_NT / 64 * K];
    __shared__ float c[K];
    cal_move<K>(from, n_wgs, scratch, c);
    if (threadIdx.x < K) out[threadIdx.x] = c[threadIdx.x];
}

template <int K>
kvq_status run_calibration(const float *x, const float *w, int64_t n, int iters, float *cent, double *partial,
                           hipStream_t s)
{
    // enough workgroups to fill the chip (three, two and one per compute unit for 4, 8 and 16 signposts, by their registers and
    // accumulators), no more than there are groups of 2048 elements, within the workspace's slots
    int64_t wgs = (n / 4 + CAL_NT - 1) / CAL_NT;
    const int64_t fill = (int64_t)kvq_cu_count() * (K == 16 ? 1 : K == 8 ? 2 : 3);
    if (wgs > fill) wgs = fill;
    if (wgs > CAL_MAX_WGS) wgs = CAL_MAX_WGS;
    if (wgs < 1) wgs = 1;
    const CalState state[2] = {{cent, partial}, {cent + 16, partial + (int64_t)CAL_MAX_WGS * 16 * 2}};
    auto run = [&](auto look_up) {
        for (int it = 0; it < iters; ++it)
            kvq_calib_assign<K, decltype(look_up)::value><<<(unsigned)wgs, CAL_NT, 0, s>>>(x, w, n, it ? (int)wgs : 0, state[it & 1],
                                                                                       state[(it + 1) & 1]);
    };
    // The look-up saves the search's four instructions per signpost and element and costs 2 us per iteration for the
    // thresholds and the workgroups' cells.  Whole calls of 20 iterations, us, look-up against search: 16 signposts, 100000
    // elements 216 / 177, 1 M 232 / 201, 4.2 M 291 / 319; 8 signposts, 1 M 232 / 188, 16.8 M 561 / 538; 4 signposts, 16.8 M 532 / 509.
    if constexpr (K == 16) {
        if (n >= CAL_LOOK_UP_MIN) run(std::true_type{});
        else run(std::false_type{});
    } else {
        run(std::false_type{});
    }
    if (iters > 0) kvq_calib_finish<K><<<1, CAL_NT, 0, s>>>((int)wgs, state[iters & 1], cent + 32);
    KVQ_HIP_CHECK(hipGetLastError());
    return KVQ_OK;
}

}  // namespace

extern "C" int64_t kvq_calibrate_workspace_bytes(void)
{
    return (int64_t)CAL_MAX_WGS * 2 * 16 * 2 * (int64_t)sizeof(double) + 256;
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
    float *cent = (float *)d_workspace;                       // twice 16 signposts and the result, then the partial sums
    double *partial = (double *)((char *)d_workspace + 256);
    KVQ_HIP_CHECK(hipMemcpyAsync(cent, h_signposts, (size_t)K * sizeof(float), hipMemcpyHostToDevice, s));
    kvq_status st = (bits == 2)   ? run_calibration<4>(d_x_norm, d_w, n, iters, cent, partial, s)
                    : (bits == 3) ? run_calibration<8>(d_x_norm, d_w, n, iters, cent, partial, s)
                                  : run_calibration<16>(d_x_norm, d_w, n, iters, cent, partial, s);
    if (st != KVQ_OK) return st;
    KVQ_HIP_CHECK(hipMemcpyAsync(h_signposts, iters > 0 ? cent + 32 : cent, (size_t)K * sizeof(float), hipMemcpyDeviceToHost, s));
    KVQ_HIP_CHECK(hipStreamSynchronize(s));
    std::sort(h_signposts, h_signposts + K);
    return KVQ_OK;
}
