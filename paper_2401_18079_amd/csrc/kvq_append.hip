// Online quantize-and-append of new Key / Value vectors (paper Sec. 3.1, 3.4, 3.6, 3.7).
//
// One workgroup per new token.  Every fp32 step is a single explicitly rounded operation
// (this file is compiled with floating-point contraction off) so that codes, outlier indices
// and fp16 residuals are reproducible bit for bit.
#include "kvq_common.hpp"
#include "kvq_qk_sparse.hpp"
#include "kvq_append_common.hpp"
#include <type_traits>

namespace {

// Launch rules.  Keys: a wavefront per token from KVQ_WAVE_TOKENS tokens on, twice that above 16 heads (3 bits, 32 heads:
// 4096 tokens 30 us against 38 us with sixteen wavefronts per token, 2500 tokens 24 / 25, 1500 tokens 22 / 17; 8 heads:
// 1500 tokens 7.2 / 9.1), sixteen wavefronts per token below (one token of 5120 channels: 10.9 us with the looping body, 5.7 us;
// 777 tokens, 4 bits: 19.9 us with 256 threads per token, 17.2 us).  Values: v_quant_token4 keeps a token in registers.
// In calls of fewer than KVQ_VW_SMALL_TOKENS tokens it takes every multiple of 1024 channels up to 8192 (small_width;
// both appends of one token, 4 bits, us with the routine for any width and with it: 24 heads 12.2 / 8.8, 48 heads
// 27.6 / 12.4, 64 heads 33.2 / 13.2; 63 tokens of 64 heads 43.7 / 25.8), one token per workgroup (two would lengthen the
// one chain that counts).  In longer calls a workgroup takes the two tokens that share dwords: kvq_v_pair.hip (see append_v), or, where
// that does not apply, four wavefronts each: 1024, 2048 and 4096 channels, and 5120, 6656 and 8192 from KVQ_BULK_TOKENS
// tokens on (4096 tokens of 4096: 74 us with a token's bits merged into memory by two atomics per dword, 51 us with whole
// dwords stored).  All others take the routine for any width.
constexpr int KVQ_BULK_TOKENS = 512;      // calls with at least this many tokens count as bulk appends
constexpr int KVQ_KV_SPLIT_TOKENS = 256;  // from here on the combined call runs the Key and Value kernels in turn,
constexpr int KVQ_KV_SPLIT_BULK = 129;    // from here on where they are those of multiples of 1024 channels, 3072 and more,
constexpr int KVQ_KV_SPLIT_NARROW = 150;  // and from here on with 1024 or 2048 channels and 2 bits
constexpr int KVQ_WAVE_TOKENS = 1024;     // Key appends of at least this many tokens: one wavefront per token

// Workgroups have NT threads: 256 for narrow models, 1024 once a token vector has >= 2048 channels
// (fewer passes over the vector, hence fewer barriers, for the single-token decode append).

// The signposts in LDS, for the residuals of outliers (a dynamic index).  The caller's next barrier makes them visible.
template <int NE>
__device__ __forceinline__ void stage_lut(float *lut_s, const float *lut)
{
    if (threadIdx.x < NE) lut_s[threadIdx.x] = lut[threadIdx.x];
}

// Exclusive rank of this thread's flag among all flags of the workgroup, in thread order, plus
// the workgroup total.  `wave_tot` is a shared array of NT/64 words.  Contains two barriers.
template <int NT>
__device__ inline uint32_t block_rank(bool flag, uint32_t *wave_tot, uint32_t &total)
{
    constexpr int NW = NT / 64;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    unsigned long long b = __ballot(flag);
    uint32_t prefix = __popcll(b & ((1ull << lane) - 1ull));
    if (lane == 0) wave_tot[w] = __popcll(b);
    __syncthreads();
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        uint32_t t = wave_tot[i];
        if (i < w) before += t;
        tot += t;
    }
    __syncthreads();
    total = tot;
    return before + prefix;
}

template <bool PACKED>
__global__ __launch_bounds__(KVQ_COUNT_NT) void kvq_k_count(const void *params, int D, int T, const uint16_t *k_new,
                                                            uint32_t *cnt)
{
    const int t = blockIdx.x * (KVQ_COUNT_NT / 64) + (threadIdx.x >> 6);
    if (t < T) k_count_token<PACKED>(params, D, k_new, cnt, t);
}

// ptr[n0+1+t] = min(ptr[n0] + cnt[0] + ... + cnt[t], cap_nnz); one workgroup, T <= 4096.
__global__ __launch_bounds__(1024) void kvq_ptr_scan(uint32_t *ptr, int64_t n0, int T, const uint32_t *cnt,
                                                     int64_t cap_nnz, int32_t *d_status)
{
    __shared__ uint32_t part[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t v[4], s = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        int t = tid * 4 + j;
        v[j] = (t < T) ? cnt[t] : 0u;
        s += v[j];
    }
    const uint64_t first = ptr[n0];
    // sums over the wavefront's lanes up to this one, then over the wavefronts before: one barrier
    uint32_t sum = s;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t add = __shfl_up(sum, o);
        sum += lane >= o ? add : 0u;
    }
    if (lane == 63) part[wave] = sum;
    __syncthreads();
    uint64_t run = first + (sum - s);
#pragma unroll
    for (int w = 0; w < 16; ++w) run += w < wave ? part[w] : 0u;
    bool over = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        int t = tid * 4 + j;
        run += v[j];
        if (t < T) {
            uint64_t p = run;
            if (p > (uint64_t)cap_nnz) { p = (uint64_t)cap_nnz; over = true; }
            ptr[n0 + 1 + t] = (uint32_t)p;
        }
    }
    if (over) atomicExch(d_status, (int32_t)KVQ_ERR_NNZ_OVERFLOW);
}

// OR one field of `width` bits into a little-endian bit stream held as dwords in shared memory.
__device__ inline void stream_or(uint32_t *words, int bit, uint32_t value, int width)
{
    int w = bit >> 5, sh = bit & 31;
    atomicOr(&words[w], value << sh);
    if (sh + width > 32) atomicOr(&words[w + 1], value >> (32 - sh));
}

// Exclusive ranks, in channel order, of IT flags per thread (flag j belongs to channel block j, a
// block being NT consecutive channels, one per thread): rank[j] counts the set flags of all earlier
// blocks plus those of lower threads in block j.  `wave_tot` is a shared array of IT*NT/64 words.
// Returns the total.  Contains two barriers, whatever IT.
template <int NT, int IT>
__device__ inline uint32_t block_rank_multi(const bool (&flag)[IT], uint32_t (&rank)[IT], uint32_t *wave_tot)
{
    constexpr int NW = NT / 64;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t prefix[IT];
#pragma unroll
    for (int j = 0; j < IT; ++j) {
        const unsigned long long b = __ballot(flag[j]);
        prefix[j] = __popcll(b & ((1ull << lane) - 1ull));
        if (lane == 0) wave_tot[j * NW + w] = __popcll(b);
    }
    __syncthreads();
    uint32_t run = 0;
#pragma unroll
    for (int j = 0; j < IT; ++j) {
        uint32_t before = 0, tot = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const uint32_t t = wave_tot[j * NW + i];
            if (i < w) before += t;
            tot += t;
        }
        rank[j] = run + before + prefix[j];
        run += tot;
    }
    __syncthreads();
    return run;
}

// Quantize, pack and append the Keys of one new token per workgroup.
// If `single` the token's outlier count is written to ptr[n+1] here; otherwise ptr[] was already
// filled by kvq_ptr_scan and is only read.
// A pass handles IT blocks of NT channels: all its loads are issued up front, and ranks, packing and
// stores of the IT blocks share one set of barriers (a single-token decode append is pure latency).
// (The body of the kernels below: `t` is the token's index within the call.)
template <int BITS, int NT, class SP>
__device__ __forceinline__ void k_quant_token(const void *__restrict__ params, int D, int64_t cap, int64_t n0,
                                              const uint16_t *__restrict__ k_new, uint8_t *__restrict__ k_codes,
                                              uint32_t *__restrict__ k_ptr, const SP ksp, int64_t cap_nnz, int single,
                                              int32_t *d_status, const int t)
{
    constexpr int NE = 1 << BITS;
    constexpr int CW = 4 * BITS;                 // dwords per chunk
    constexpr int NW = NT / 64;
    constexpr int HB = NT / KVQ_HEAD_DIM;        // heads covered by one block of NT channels
    constexpr int IT = 4;                        // blocks per pass
    __shared__ uint8_t codes_s[IT][NT];
    __shared__ uint32_t chunk_s[IT][HB][CW + 1];
    __shared__ uint32_t wave_tot[IT * NW];
    KvqParamsView pv = kvq_params_view(params, D);
    __shared__ float lut_s[NE];
    const KvqCoder<NE> coder(pv.hdr->thr_k, pv.hdr->lut_k);
    stage_lut<NE>(lut_s, pv.hdr->lut_k);
    __syncthreads();

    const int tid = threadIdx.x;
    const int64_t n = n0 + t;
    const uint32_t base = k_ptr[n];
    uint32_t running = 0;
    bool overflow = false;
    for (int cb = 0; cb < D; cb += NT * IT) {
        bool is_out[IT];
        uint16_t resid[IT];
        // every load of the pass first (no short-circuit evaluation below: a conditional load would
        // wait for the ones before it), then the arithmetic
        uint16_t xb[IT];
        float zc[IT], sc[IT], ri[IT], lo[IT], hi[IT];
#pragma unroll
        for (int j = 0; j < IT; ++j) {
            const int c = cb + j * NT + tid;
            const int cc = (c < D) ? c : D - 1;                      // clamped: straight-line loads
            xb[j] = k_new[(int64_t)t * D + cc];
            zc[j] = pv.z[cc]; sc[j] = pv.s[cc]; ri[j] = pv.rinv[cc]; lo[j] = pv.lo[cc]; hi[j] = pv.hi[cc];
        }
#pragma unroll
        for (int j = 0; j < IT; ++j) {
            const int c = cb + j * NT + tid;
            const float x = kvq_h2f(xb[j]);
            const float diff = x - zc[j];
            const float xn = diff * ri[j];
            const int code = coder(xn);
            is_out[j] = (c < D) & ((x < lo[j]) | (x > hi[j]));
            resid[j] = 0;
            if (is_out[j]) resid[j] = kvq_f2h_rn(x - __builtin_fmaf(sc[j], lut_s[code], zc[j]));
            codes_s[j][tid] = (uint8_t)code;
        }
        for (int i = tid; i < IT * HB * (CW + 1); i += NT) (&chunk_s[0][0][0])[i] = 0;
        uint32_t rank[IT];
        const uint32_t tot = block_rank_multi<NT, IT>(is_out, rank, wave_tot);   // barriers inside
#pragma unroll
        for (int j = 0; j < IT; ++j) {
            if (is_out[j]) {
                const uint64_t pos = (uint64_t)base + running + rank[j];
                if (pos < (uint64_t)cap_nnz) ksp.put(pos, (uint16_t)(cb + j * NT + tid), resid[j]);
                else overflow = true;
            }
        }
        running += tot;
        // pack the heads covered by each block of NT channels
#pragma unroll
        for (int j = 0; j < IT; ++j) {
            const int c0 = cb + j * NT;
            const int heads_here = (c0 >= D) ? 0 : ((D - c0 >= NT) ? HB : (D - c0) / KVQ_HEAD_DIM);
            if (tid < 64 * heads_here) {
                const int hh = tid >> 6, i = tid & 63;
                const uint32_t field = (uint32_t)codes_s[j][hh * 128 + i] | ((uint32_t)codes_s[j][hh * 128 + i + 64] << BITS);
                stream_or(chunk_s[j][hh], i * 2 * BITS, field, 2 * BITS);
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < IT; ++j) {
            const int c0 = cb + j * NT;
            const int heads_here = (c0 >= D) ? 0 : ((D - c0 >= NT) ? HB : (D - c0) / KVQ_HEAD_DIM);
            if (tid < CW * heads_here) {
                const int hh = tid / CW, wd = tid % CW;
                const int64_t off = kvq_k_piece0(BITS, cap, n, c0 / KVQ_HEAD_DIM + hh) + (wd >> 2) * 1024 + (wd & 3) * 4;
                *(uint32_t *)(k_codes + off) = chunk_s[j][hh][wd];
            }
        }
        if (cb + NT * IT < D) __syncthreads();       // the next pass reuses the shared arrays
    }
    if (single && tid == 0) {
        uint64_t p = (uint64_t)base + running;
        k_ptr[n + 1] = (uint32_t)(p > (uint64_t)cap_nnz ? (uint64_t)cap_nnz : p);
    }
    if (overflow || (single && tid == 0 && (uint64_t)base + running > (uint64_t)cap_nnz))
        atomicExch(d_status, (int32_t)KVQ_ERR_NNZ_OVERFLOW);
}

// The same for up to W * HW heads: W wavefronts, HW heads each, one pass and one workgroup barrier.  Lane l takes
// channels l and l+64 of a head, the pair that shares a field, and a wavefront packs its heads' chunks on its
// own; outliers keep channel order (within a head the lower channels, then the upper ones) by ballots, across
// wavefronts by their counts.  A token is latency: what counts is the length of a lane's chain.  Measured (4096
// channels, 4-bit codes, one token): see the launch rule.
template <int BITS, int HW, int W, class SP>
__device__ __forceinline__ void k_quant_token_w(const void *__restrict__ params, int D, int64_t cap, int64_t n0,
                                                const uint16_t *__restrict__ k_new, uint8_t *__restrict__ k_codes,
                                                uint32_t *__restrict__ k_ptr, const SP ksp, int64_t cap_nnz, int single,
                                                int32_t *d_status, const int t)
{
    constexpr int NE = 1 << BITS;
    constexpr int CW = 4 * BITS;                 // dwords per chunk
    __shared__ uint32_t chunk_s[W][HW][CW + 1];
    __shared__ uint32_t wave_tot[W];
    __shared__ float lut_s[NE];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int H = D / KVQ_HEAD_DIM, h0 = wave * HW;
    const KvqParamsView pv = kvq_params_view(params, D);
    const int64_t n = n0 + t;
    const uint32_t base = k_ptr[n];
    // every load first; heads past the last one repeat it and store nothing
    uint16_t xb[HW][2];
    float z[HW][2], sc[HW][2], ri[HW][2], lo[HW][2], hi[HW][2];
#pragma unroll
    for (int i = 0; i < HW; ++i)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int h = h0 + i < H ? h0 + i : H - 1, c = h * KVQ_HEAD_DIM + 64 * u + lane;
            xb[i][u] = k_new[(int64_t)t * D + c];
            z[i][u] = pv.z[c]; sc[i][u] = pv.s[c]; ri[i][u] = pv.rinv[c]; lo[i][u] = pv.lo[c]; hi[i][u] = pv.hi[c];
        }
    const KvqCoder<NE> coder(pv.hdr->thr_k, pv.hdr->lut_k);
    stage_lut<NE>(lut_s, pv.hdr->lut_k);
    for (int e = lane; e < HW * (CW + 1); e += 64) (&chunk_s[wave][0][0])[e] = 0;
    uint32_t mine = 0;
    bool out[HW][2];
#pragma unroll
    for (int i = 0; i < HW; ++i)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const float x = kvq_h2f(xb[i][u]);
            out[i][u] = (h0 + i < H) & ((x < lo[i][u]) | (x > hi[i][u]));
            mine += (uint32_t)__popcll(__ballot(out[i][u]));
        }
    if (lane == 0) wave_tot[wave] = mine;
    __syncthreads();
    uint32_t running = 0, total = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const uint32_t c = wave_tot[w];
        running += w < wave ? c : 0u;
        total += c;
    }
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    bool overflow = false;
#pragma unroll
    for (int i = 0; i < HW; ++i) {
        if (h0 + i >= H) break;
        int code[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const float x = kvq_h2f(xb[i][u]);
            const float diff = x - z[i][u];
            code[u] = coder(diff * ri[i][u]);
            const unsigned long long b = __ballot(out[i][u]);
            if (out[i][u]) {
                const uint64_t pos = (uint64_t)base + running + (uint32_t)__popcll(b & lt_mask);
                if (pos < (uint64_t)cap_nnz)
                    ksp.put(pos, (uint16_t)((h0 + i) * KVQ_HEAD_DIM + 64 * u + lane),
                            kvq_f2h_rn(x - __builtin_fmaf(sc[i][u], lut_s[code[u]], z[i][u])));
                else overflow = true;
            }
            running += (uint32_t)__popcll(b);
        }
        stream_or(chunk_s[wave][i], lane * 2 * BITS, (uint32_t)code[0] | ((uint32_t)code[1] << BITS), 2 * BITS);
    }
    // LDS operations of one wavefront execute in order; the fence keeps the compiler from reordering them
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int e = lane; e < HW * CW; e += 64) {
        const int i = e / CW, wd = e - i * CW;
        if (h0 + i < H)
            *(uint32_t *)(k_codes + kvq_k_piece0(BITS, cap, n, h0 + i) + (wd >> 2) * 1024 + (wd & 3) * 4) = chunk_s[wave][i][wd];
    }
    const uint64_t end = (uint64_t)base + total;
    if (single && threadIdx.x == 0) k_ptr[n + 1] = (uint32_t)(end > (uint64_t)cap_nnz ? (uint64_t)cap_nnz : end);
    if (overflow || (single && threadIdx.x == 0 && end > (uint64_t)cap_nnz))
        atomicExch(d_status, (int32_t)KVQ_ERR_NNZ_OVERFLOW);
}

// ---- Values -------------------------------------------------------------------------------

// For the 256 histogram bins held one per thread (threads >= 256 pass 0): the number of elements in
// bins strictly above this thread's bin.  Suffix scan inside each wavefront plus the totals of the
// (up to four) wavefronts that hold bins.  `wsum` is a shared array of 4 words.  One barrier.
__device__ inline uint32_t bins_above(uint32_t mine, uint32_t *wsum)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t s = mine;                            // becomes the sum over lanes lane..63
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_down(s, o);
        if (lane + o < 64) s += t;
    }
    if (lane == 0 && w < 4) wsum[w] = s;
    __syncthreads();
    uint32_t above = s - mine;
    for (int i = w + 1; i < 4; ++i) above += wsum[i];
    return above;
}

// Workgroup-wide selection of the `k` largest keys among elements with state[c]==0, where the key
// of element c is keys[c] ^ flip (flip = 0xFFFF turns it into a selection of the k smallest).
// Marks the selected elements with `mark`; equal keys are taken in ascending index order.
// Two-level radix select on the 16-bit keys; the index-ordered pass over the elements equal to the
// threshold is only needed when some but not all of them are taken.
template <int NT>
__device__ void select_top(const uint16_t *keys, uint8_t *state, int D, int k, uint32_t flip, uint8_t mark,
                           uint32_t *hist, uint32_t *sh, uint32_t *wave_tot)
{
    const int tid = threadIdx.x;
    // level 1: high byte
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    for (int c = tid; c < D; c += NT)
        if (state[c] == 0) atomicAdd(&hist[((keys[c] ^ flip) & 0xFFFFu) >> 8], 1u);
    __syncthreads();
    {
        const uint32_t mine = (tid < 256) ? hist[tid] : 0u;
        const uint32_t above = bins_above(mine, sh + 4);      // elements in bins strictly above bin `tid`
        if (tid < 256 && above < (uint32_t)k && above + mine >= (uint32_t)k) { sh[0] = tid; sh[1] = above; }
    }
    __syncthreads();
    const uint32_t bin_hi = sh[0], above_hi = sh[1];
    __syncthreads();
    // level 2: low byte inside the selected high bin
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    for (int c = tid; c < D; c += NT) {
        uint32_t key = (keys[c] ^ flip) & 0xFFFFu;
        if (state[c] == 0 && (key >> 8) == bin_hi) atomicAdd(&hist[key & 255u], 1u);
    }
    __syncthreads();
    {
        const uint32_t mine = (tid < 256) ? hist[tid] : 0u;
        const uint32_t above = above_hi + bins_above(mine, sh + 4);
        if (tid < 256 && above < (uint32_t)k && above + mine >= (uint32_t)k) {
            sh[0] = (bin_hi << 8) | tid; sh[1] = above; sh[2] = mine;
        }
    }
    __syncthreads();
    const uint32_t tau = sh[0];
    const uint32_t need_eq = (uint32_t)k - sh[1];  // how many elements equal to tau are taken
    const bool all_eq = need_eq == sh[2];          // ... all of them: no index order needed
    __syncthreads();
    if (all_eq) {
        for (int c = tid; c < D; c += NT)
            if (state[c] == 0 && ((keys[c] ^ flip) & 0xFFFFu) >= tau) state[c] = mark;
    } else {
        uint32_t running = 0;
        for (int c0 = 0; c0 < D; c0 += NT) {
            const int c = c0 + tid;
            bool cand = false, eq = false, gt = false;
            if (c < D && state[c] == 0) {
                uint32_t key = (keys[c] ^ flip) & 0xFFFFu;
                gt = key > tau;
                eq = key == tau;
                cand = true;
            }
            uint32_t tot;
            uint32_t rank = running + block_rank<NT>(eq, wave_tot, tot);
            running += tot;
            if (cand && (gt || (eq && rank < need_eq))) state[c] = mark;
        }
    }
    __syncthreads();
}

// Two bin sets at once (same scan as bins_above, one barrier for both).  `wsum` holds 8 words.
__device__ inline void bins_above2(uint32_t mine_a, uint32_t mine_b, uint32_t *wsum, uint32_t &above_a,
                                   uint32_t &above_b)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t sa = mine_a, sb = mine_b;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t ta = __shfl_down(sa, o), tb = __shfl_down(sb, o);
        if (lane + o < 64) { sa += ta; sb += tb; }
    }
    if (lane == 0 && w < 4) { wsum[w] = sa; wsum[4 + w] = sb; }
    __syncthreads();
    above_a = sa - mine_a;
    above_b = sb - mine_b;
    for (int i = w + 1; i < 4; ++i) { above_a += wsum[i]; above_b += wsum[4 + i]; }
}

// The k largest keys (marked 1) and, among the rest, the k smallest (marked 2) in one go; state[] is
// all zero on entry and 2k < D.  Equal keys are taken in ascending index order on both sides.  Both
// thresholds come out of the same two histogram passes (high byte, then low byte inside the two
// selected bins).  Because 2k < D the k-th largest key is >= the k-th smallest; when they differ the
// two selections cannot interact and this routine is exact; when they coincide (heavy ties) it
// leaves state[] untouched and returns false, and the caller runs the two selections one after the
// other.  hist: 768 words that the caller has cleared (and made visible with a barrier), sh: 24
// words, wave_tot: 2*NT/64 words.
template <int NT>
__device__ bool select_both(const uint16_t *keys, uint8_t *state, int D, int k, uint32_t *hist, uint32_t *sh,
                            uint32_t *wave_tot)
{
    const int tid = threadIdx.x;
    const uint32_t K = (uint32_t)k;
    for (int c = tid; c < D; c += NT) atomicAdd(&hist[keys[c] >> 8], 1u);
    __syncthreads();
    {
        const uint32_t mine = (tid < 256) ? hist[tid] : 0u;
        const uint32_t above = bins_above(mine, sh + 16);
        const uint32_t below = (uint32_t)D - above - mine;
        if (tid < 256 && above < K && above + mine >= K) { sh[0] = tid; sh[1] = above; }
        if (tid < 256 && below < K && below + mine >= K) { sh[2] = tid; sh[3] = below; sh[4] = mine; }
    }
    __syncthreads();
    const uint32_t bin_top = sh[0], above_top = sh[1], bin_bot = sh[2], below_bot = sh[3], in_bot = sh[4];
    for (int c = tid; c < D; c += NT) {
        const uint32_t key = keys[c];
        if ((key >> 8) == bin_top) atomicAdd(&hist[256 + (key & 255u)], 1u);
        if ((key >> 8) == bin_bot) atomicAdd(&hist[512 + (key & 255u)], 1u);
    }
    __syncthreads();
    {
        const uint32_t mt = (tid < 256) ? hist[256 + tid] : 0u, mb = (tid < 256) ? hist[512 + tid] : 0u;
        uint32_t at, ab;
        bins_above2(mt, mb, sh + 16, at, ab);
        const uint32_t above = above_top + at;                   // keys strictly greater than this one
        const uint32_t below = below_bot + (in_bot - ab - mb);   // keys strictly smaller than this one
        if (tid < 256 && above < K && above + mt >= K) { sh[5] = (bin_top << 8) | tid; sh[6] = above; sh[7] = mt; }
        if (tid < 256 && below < K && below + mb >= K) { sh[8] = (bin_bot << 8) | tid; sh[9] = below; sh[10] = mb; }
    }
    __syncthreads();
    const uint32_t tau_top = sh[5], tau_bot = sh[8];
    const uint32_t need_top = K - sh[6], need_bot = K - sh[9];
    const bool all_top = need_top == sh[7], all_bot = need_bot == sh[10];
    if (tau_top == tau_bot) return false;
    if (all_top && all_bot) {
        for (int c = tid; c < D; c += NT) {
            const uint32_t key = keys[c];
            if (key >= tau_top) state[c] = 1;
            else if (key <= tau_bot) state[c] = 2;
        }
    } else {
        // ties straddle a threshold: equal keys are taken in index order
        uint32_t run_top = 0, run_bot = 0;
        for (int c0 = 0; c0 < D; c0 += NT) {
            const int c = c0 + tid;
            const uint32_t key = (c < D) ? keys[c] : 0u;
            const bool flag[2] = {c < D && key == tau_top, c < D && key == tau_bot};
            uint32_t rank[2];
            // ranks of flag[1] continue after all of flag[0]: take the per-flag counts apart again
            const uint32_t both = block_rank_multi<NT, 2>(flag, rank, wave_tot);
            const uint32_t n_top = __syncthreads_count(flag[0]);
            const uint32_t rt = run_top + rank[0], rb = run_bot + (rank[1] - n_top);
            if (c < D) {
                if (key > tau_top || (flag[0] && rt < need_top)) state[c] = 1;
                else if (key < tau_bot || (flag[1] && rb < need_bot)) state[c] = 2;
            }
            run_top += n_top;
            run_bot += both - n_top;
        }
    }
    __syncthreads();
    return true;
}

// Quantize, pack and append the Values of one new token per workgroup (`t`: the token's index within
// the call).  A pass of the main loop handles IT blocks of NT channels (see k_quant_token).
template <int BITS, int NT, class SP>
__device__ __forceinline__ void v_quant_token(const void *__restrict__ params, int D, int64_t cap, int64_t n0,
                                              int k_side, const uint16_t *__restrict__ v_new,
                                              uint8_t *__restrict__ v_codes, uint16_t *__restrict__ v_sz,
                                              uint32_t *__restrict__ v_ptr, const SP vsp, int64_t cap_nnz, int32_t *d_status,
                                              const int t)
{
    constexpr int NE = 1 << BITS;
    constexpr int CW = 4 * BITS;
    constexpr int IT = 4;                         // blocks per pass
    extern __shared__ uint8_t dyn[];              // keys: 2*D bytes, state: D bytes
    uint16_t *keys = (uint16_t *)dyn;
    uint8_t *state = dyn + 2 * (size_t)D;
    constexpr int NW = NT / 64;
    constexpr int CB = NT / 64;                   // (head, half) chunks covered by one block of NT channels
    __shared__ uint32_t hist[768];
    __shared__ uint32_t sh[24];
    __shared__ uint32_t wave_tot[IT * NW];
    __shared__ float redmx[NW], redmn[NW];
    __shared__ uint8_t codes_s[IT][NT];
    __shared__ uint32_t bits_s[IT][CB][CW + 1], mask_s[IT][CB][CW + 1];

    __shared__ float lut_s[NE];
    KvqParamsView pv = kvq_params_view(params, D);
    const KvqCoder<NE> coder(pv.hdr->thr_v, pv.hdr->lut_v);
    stage_lut<NE>(lut_s, pv.hdr->lut_v);             // (visible after the barriers of the selection)
    const int tid = threadIdx.x;
    const int64_t n = n0 + t;
    const uint16_t *x16 = v_new + (int64_t)t * D;
    const uint32_t base = v_ptr[n0] + (uint32_t)t * 2u * (uint32_t)k_side;

    // The thread's first IT elements (channels tid, tid + NT, ...) stay in registers for the later
    // passes; wider vectors re-read the rest from memory.
    uint16_t xc[IT];
#pragma unroll
    for (int j = 0; j < IT; ++j) {
        const int c = tid + j * NT;
        xc[j] = x16[c < D ? c : D - 1];
    }
#pragma unroll
    for (int j = 0; j < IT; ++j) {
        const int c = tid + j * NT;
        if (c < D) { keys[c] = (uint16_t)order_key(xc[j]); state[c] = 0; }
    }
    for (int c = tid + IT * NT; c < D; c += NT) { keys[c] = (uint16_t)order_key(x16[c]); state[c] = 0; }
    for (int i = tid; i < 768; i += NT) hist[i] = 0;   // the three histograms of select_both
    __syncthreads();
    if (k_side > 0) {
        if (!select_both<NT>(keys, state, D, k_side, hist, sh, wave_tot)) {
            select_top<NT>(keys, state, D, k_side, 0u, 1, hist, sh, wave_tot);        // k largest
            select_top<NT>(keys, state, D, k_side, 0xFFFFu, 2, hist, sh, wave_tot);   // k smallest of the rest
        }
    }
    // range of the remaining elements
    float mx = -INFINITY, mn = INFINITY;
#pragma unroll
    for (int j = 0; j < IT; ++j) {
        const int c = tid + j * NT;
        if (c < D && state[c] == 0) { float x = kvq_h2f(xc[j]); mx = fmaxf(mx, x); mn = fminf(mn, x); }
    }
    for (int c = tid + IT * NT; c < D; c += NT)
        if (state[c] == 0) { float x = kvq_h2f(x16[c]); mx = fmaxf(mx, x); mn = fminf(mn, x); }
    for (int o = 32; o > 0; o >>= 1) { mx = fmaxf(mx, __shfl_xor(mx, o)); mn = fminf(mn, __shfl_xor(mn, o)); }
    if ((tid & 63) == 0) { redmx[tid >> 6] = mx; redmn[tid >> 6] = mn; }
    __syncthreads();
    mx = redmx[0]; mn = redmn[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) { mx = fmaxf(mx, redmx[i]); mn = fminf(mn, redmn[i]); }
    const float sum = mx + mn, dif = mx - mn;
    uint16_t zb = kvq_f2h_rn(sum * 0.5f), sb = kvq_f2h_rn(dif * 0.5f);
    float zf = kvq_h2f(zb), sf = kvq_h2f(sb);
    if (sf == 0.0f) { sf = 1.0f; sb = 0x3c00u; }
    const float rinv = __fdiv_rn(1.0f, sf);
    if (tid == 0) { v_sz[n * 2 + 0] = sb; v_sz[n * 2 + 1] = zb; }

    const int parity = (int)(n & 1);
    uint32_t running = 0;
    bool overflow = false;
    for (int cb = 0; cb < D; cb += NT * IT) {
        bool is_out[IT];
        uint16_t resid[IT];
#pragma unroll
        for (int j = 0; j < IT; ++j) {
            const int c = cb + j * NT + tid;
            const int cc = (c < D) ? c : D - 1;
            const float x = kvq_h2f(cb == 0 ? xc[j] : x16[cc]);      // the first pass has its elements in registers
            const float diff = x - zf;
            const float xn = diff * rinv;
            const int code = coder(xn);
            is_out[j] = (c < D) && state[cc] != 0;
            resid[j] = 0;
            if (is_out[j]) resid[j] = kvq_f2h_rn(x - __builtin_fmaf(sf, lut_s[code], zf));
            codes_s[j][tid] = (uint8_t)code;
        }
        for (int i = tid; i < IT * CB * (CW + 1); i += NT) { (&bits_s[0][0][0])[i] = 0; (&mask_s[0][0][0])[i] = 0; }
        uint32_t rank[IT];
        const uint32_t tot = block_rank_multi<NT, IT>(is_out, rank, wave_tot);   // barriers inside
#pragma unroll
        for (int j = 0; j < IT; ++j) {
            if (is_out[j]) {
                const uint64_t pos = (uint64_t)base + running + rank[j];
                if (pos < (uint64_t)cap_nnz) vsp.put(pos, (uint16_t)(cb + j * NT + tid), resid[j]);
                else overflow = true;
            }
        }
        running += tot;
        // a block of NT channels covers up to CB (head, half) chunks of 64 fields each
#pragma unroll
        for (int j = 0; j < IT; ++j) {
            const int c0 = cb + j * NT;
            const int chunks_here = (c0 >= D) ? 0 : ((D - c0 >= NT) ? CB : (D - c0) / 64);
            if (tid < 64 * chunks_here) {
                const int q = tid >> 6, i = tid & 63;
                stream_or(bits_s[j][q], i * 2 * BITS + parity * BITS, (uint32_t)codes_s[j][tid], BITS);
                stream_or(mask_s[j][q], i * 2 * BITS + parity * BITS, (uint32_t)(NE - 1), BITS);
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < IT; ++j) {
            const int c0 = cb + j * NT;
            const int chunks_here = (c0 >= D) ? 0 : ((D - c0 >= NT) ? CB : (D - c0) / 64);
            if (tid < CW * chunks_here) {
                const int q = tid / CW, wd = tid % CW;
                const int ch0 = c0 + q * 64;
                const int64_t off = kvq_v_piece0(BITS, cap, n >> 1, ch0 / KVQ_HEAD_DIM, (ch0 >> 6) & 1) + (wd >> 2) * 1024 + (wd & 3) * 4;
                uint32_t *p = (uint32_t *)(v_codes + off);
                // The partner token of the pair owns the other bits of this dword and may be written
                // concurrently by another workgroup: clear this token's bits, then set them, with two
                // atomics that return nothing (no round trip; the same thread's atomics on one address
                // are applied in order, and the partner's touch disjoint bits).
                __hip_atomic_fetch_and(p, ~mask_s[j][q][wd], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_fetch_or(p, bits_s[j][q][wd], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (cb + NT * IT < D) __syncthreads();     // the next pass reuses the shared arrays
    }
    if (tid == 0) {
        uint64_t p = (uint64_t)base + 2u * (uint32_t)k_side;
        if (p > (uint64_t)cap_nnz) { p = (uint64_t)cap_nnz; overflow = true; }
        v_ptr[n + 1] = (uint32_t)p;
    }
    if (overflow) atomicExch(d_status, (int32_t)KVQ_ERR_NNZ_OVERFLOW);
}

// Bulk Key append: one wavefront per token, no workgroup barrier.  Lane l takes channels l and l+64
// of every head, the pair that shares a field of the packed chunk, so a head's 64 fields come from the
// 64 lanes; the chunk is assembled in a slice of LDS private to the wavefront.  Outliers keep channel
// order: within a head first the lanes' lower channels, then their upper ones, ranked by ballots.
// Same arithmetic, same results, as k_quant_token; the per-token pointers come from kvq_ptr_scan.
constexpr int KVQ_KW_NT = 256;
template <int BITS, class SP>
__global__ __launch_bounds__(KVQ_KW_NT) void kvq_k_quant_wave(const void *__restrict__ params, int D, int T,
                                                              int64_t cap, int64_t n0,
                                                              const uint16_t *__restrict__ k_new,
                                                              uint8_t *__restrict__ k_codes,
                                                              const uint32_t *__restrict__ k_ptr,
                                                              const SP ksp, int64_t cap_nnz,
                                                              int32_t *d_status)
{
    constexpr int NE = 1 << BITS;
    constexpr int CW = 4 * BITS;                 // dwords per chunk
    __shared__ uint32_t chunk_s[KVQ_KW_NT / 64][CW + 1];
    __shared__ float lut_s[NE];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t = blockIdx.x * (KVQ_KW_NT / 64) + wave;
    KvqParamsView pv = kvq_params_view(params, D);
    const KvqCoder<NE> coder(pv.hdr->thr_k, pv.hdr->lut_k);
    stage_lut<NE>(lut_s, pv.hdr->lut_k);
    __syncthreads();
    if (t >= T) return;                          // whole wavefronts leave; there is no workgroup barrier below
    const int64_t n = n0 + t;
    const uint32_t base = k_ptr[n];
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    uint32_t *chunk = chunk_s[wave];
    uint32_t running = 0;
    bool overflow = false;
    const int H = D / KVQ_HEAD_DIM;
    for (int h = 0; h < H; ++h) {
        const int c0 = h * KVQ_HEAD_DIM + lane, c1 = c0 + 64;
        const uint16_t xb0 = k_new[(int64_t)t * D + c0], xb1 = k_new[(int64_t)t * D + c1];
        const float z0 = pv.z[c0], s0 = pv.s[c0], r0 = pv.rinv[c0], lo0 = pv.lo[c0], hi0 = pv.hi[c0];
        const float z1 = pv.z[c1], s1 = pv.s[c1], r1 = pv.rinv[c1], lo1 = pv.lo[c1], hi1 = pv.hi[c1];
        if (lane <= CW) chunk[lane] = 0;
        const float x0 = kvq_h2f(xb0), x1 = kvq_h2f(xb1);
        const float d0 = x0 - z0, d1 = x1 - z1;
        const float xn0 = d0 * r0, xn1 = d1 * r1;
        int code0 = coder.count(xn0), code1 = coder.count(xn1);
        if (__ballot(coder.far(xn0) | coder.far(xn1)) != 0ull) {
            if (coder.far(xn0)) code0 = coder.search(xn0);
            if (coder.far(xn1)) code1 = coder.search(xn1);
        }
        const bool o0 = (x0 < lo0) | (x0 > hi0), o1 = (x1 < lo1) | (x1 > hi1);
        // outliers of this head in channel order
        const unsigned long long b0 = __ballot(o0), b1 = __ballot(o1);
        const uint32_t rank0 = running + (uint32_t)__popcll(b0 & lt_mask);
        running += (uint32_t)__popcll(b0);
        const uint32_t rank1 = running + (uint32_t)__popcll(b1 & lt_mask);
        running += (uint32_t)__popcll(b1);
        if (o0) {
            const uint64_t pos = (uint64_t)base + rank0;
            if (pos < (uint64_t)cap_nnz) ksp.put(pos, (uint16_t)c0, kvq_f2h_rn(x0 - __builtin_fmaf(s0, lut_s[code0], z0)));
            else overflow = true;
        }
        if (o1) {
            const uint64_t pos = (uint64_t)base + rank1;
            if (pos < (uint64_t)cap_nnz) ksp.put(pos, (uint16_t)c1, kvq_f2h_rn(x1 - __builtin_fmaf(s1, lut_s[code1], z1)));
            else overflow = true;
        }
        // the head's chunk: 64 fields of 2*BITS bits, assembled in the wavefront's LDS slice (LDS
        // operations of one wavefront execute in order; the fences keep the compiler from reordering them)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        stream_or(chunk, lane * 2 * BITS, (uint32_t)code0 | ((uint32_t)code1 << BITS), 2 * BITS);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (lane < CW) {
            const int64_t off = kvq_k_piece0(BITS, cap, n, h) + (lane >> 2) * 1024 + (lane & 3) * 4;
            *(uint32_t *)(k_codes + off) = chunk[lane];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if (overflow) atomicExch(d_status, (int32_t)KVQ_ERR_NNZ_OVERFLOW);
}

// Counts the lanes with `in` set in the bins of a histogram.  Additions to one word of LDS go one after the other:
// where a token's keys are mostly equal (`tied`), the lanes that share the first one's bin are counted in one
// addition.  64 tokens of 4096 equal channels, two per workgroup: 35 -> 23 us; done always, it costs 64 ordinary
// tokens with 65 outliers a side 5 of 17 us.
__device__ __forceinline__ void hist_count(uint32_t *hist, bool in, uint32_t bin, int lane, bool tied)
{
    if (!tied) {
        if (in) atomicAdd(&hist[bin], 1u);
        return;
    }
    const unsigned long long active = __ballot(in);
    if (active == 0ull) return;
    const int first = __ffsll(active) - 1;
    const uint32_t bin0 = (uint32_t)__builtin_amdgcn_readlane((int)bin, first);
    const unsigned long long same = __ballot(in && bin == bin0);
    if (lane == first) atomicAdd(&hist[bin0], (uint32_t)__popcll(same));
    else if (in && bin != bin0) atomicAdd(&hist[bin], 1u);
}

// The largest x below 2^(2 STEPS) that at least `rank` of the wavefront's numbers reach (N a lane), two bits at a time: the three
// questions of a step do not wait for one another.  For one wavefront alone: the steps are a chain of a ballot, a count and a choice,
// and sixteen wavefronts that all went through it took four times as long.
template <int N, int STEPS>
__device__ __forceinline__ uint32_t wave_rank(const uint32_t (&v)[N], uint32_t rank, int steps = STEPS)
{
    auto reached = [&](uint32_t x) {
        uint32_t c = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) c += (uint32_t)__popcll(__ballot(v[i] >= x));
        return c >= rank;
    };
    uint32_t x = 0;
    for (int s = steps - 1; s >= 0; --s) {
        const uint32_t d = 1u << (2 * s);
        const bool a = reached(x + d), b = reached(x + 2 * d), c = reached(x + 3 * d);
        x += c ? 3 * d : b ? 2 * d : a ? d : 0u;
    }
    return x;
}

// A number whose highest bit is that of the largest of the wavefront's.
__device__ __forceinline__ uint32_t wave_magnitude(uint32_t v)
{
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xf, 0xf, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xf, 0xf, false);
    return (uint32_t)(__builtin_amdgcn_readlane((int)v, 0) | __builtin_amdgcn_readlane((int)v, 16) |
                      __builtin_amdgcn_readlane((int)v, 32) | __builtin_amdgcn_readlane((int)v, 48));
}
// Among the wavefront's keys (N a lane; `extreme`: this lane's largest), the rank-th largest, how many of the keys equal to it are among the `rank`
// largest, and how many there are.  The rank-th largest of the lanes' extremes bounds it from below.
template <int N>
__device__ __forceinline__ void wave_threshold(const uint32_t (&key)[N], uint32_t extreme, uint32_t rank, uint32_t &tau, uint32_t &need, uint32_t &n_eq)
{
    uint32_t from = 0;
    if (N > 2 && rank <= 64u) {
        const uint32_t c[1] = {extreme};
        from = wave_rank<1, 8>(c, rank);
    }
    uint32_t v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = key[i] >= from ? key[i] - from + 1u : 0u;
    const uint32_t x = wave_rank<N, 9>(v, rank, (33 - __builtin_clz(wave_magnitude(extreme >= from ? extreme - from + 1u : 0u))) / 2);
    uint32_t beyond = 0, reached = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        beyond += (uint32_t)__popcll(__ballot(v[i] > x));
        reached += (uint32_t)__popcll(__ballot(v[i] >= x));
    }
    tau = x - 1u + from;
    need = rank - beyond;
    n_eq = reached - beyond;
}

// ---- bulk Value append -----------------------------------------------------------------------
// Value append: W wavefronts per token, D = 64 W JW channels; in bulk four (JW = 4, 8, 16, 20, 26 or 32), with two
// tokens (TOK), the pair that shares dwords, in a workgroup.  Wavefront w of a token takes the channel groups j = w JW .. (w + 1) JW - 1, lane l of it the channels
// 64 j + l (half j & 1 of head j >> 1), so a wavefront packs whole chunks on its own, channel order is
// wavefront order, and a lane keeps its JW elements in registers from the one load to the end.  The
// thresholds of the selection are found among the few keys that pass a bound (or, where these are too
// many, by a two-level radix selection on histograms shared by the wavefronts); equal keys at a threshold
// are taken in channel order, ranked with ballots and the wavefronts' counts, and when the two thresholds coincide the
// upper outliers take the first of the equal keys and the lower ones the next, which is what taking
// the k largest first and then the k smallest of the rest comes to.  The packed codes of all JW chunks
// are gathered in the wavefront's LDS slice and written by all 64 lanes at the end (whole dwords where the
// workgroup has both tokens of the pair).  Same arithmetic, same results, as
// v_quant_token.
// Calls of a few tokens take more wavefronts and one token per workgroup: fewer elements per lane, where the time of a token is the length of a lane's instruction stream
// (a 4096-channel token: 16 elements per lane on four wavefronts, 4 on sixteen).
constexpr int KVQ_VW_WAVES = 4;
constexpr int KVQ_VW_SMALL_TOKENS = 64;      // calls below this many tokens use one lane per four elements
template <int BITS, int JW, int W, int TOK, class SP>
__device__ __forceinline__ void v_quant_token4(const void *__restrict__ params, int D, int64_t cap, int64_t n0,
                                               int k_side, const uint16_t *__restrict__ v_new,
                                               uint8_t *__restrict__ v_codes, uint16_t *__restrict__ v_sz,
                                               uint32_t *__restrict__ v_ptr, const SP vsp, int64_t cap_nnz, int32_t *d_status,
                                               const int first, const int T)
{
    constexpr int NE = 1 << BITS;
    constexpr int CW = 4 * BITS;
    constexpr int NTW = 64 * W;                  // threads that work on a token
    __shared__ __attribute__((aligned(16))) uint32_t hist_s[TOK][768];
    __shared__ uint32_t bits_s[W][JW][CW + 1], mask_s[TOK][W][CW + 1];
    __shared__ uint32_t eq_cnt_s[TOK][W][2], out_cnt_s[TOK][W];
    // the largest keys of the 64 columns (lane l of every wavefront), of the keys and of their complements; the
    // candidates of either side and how many there are
    __shared__ uint32_t col_max_s[TOK][2][64], n_cand_s[TOK][2];
    __shared__ uint16_t cand_s[TOK][2][KVQ_V_CAND];
    __shared__ float red_mx_s[TOK][W], red_mn_s[TOK][W];
    // by side: the bound, as searched for; the threshold, likewise, how many candidates lie beyond it and how many equal it
    __shared__ uint32_t bound_s[TOK][2], found_s[TOK][2][3];
    // wavefronts 0 .. W-1 take the pair's first token, the next W its second; `wave`: within the token
    const int lane = threadIdx.x & 63;
    const int tok = TOK == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x / NTW));
    const int wave = (int)(threadIdx.x >> 6) - tok * W, ttid = (int)threadIdx.x - tok * NTW;
    uint32_t *hist = hist_s[tok];
    uint32_t(*eq_cnt)[2] = eq_cnt_s[tok];
    uint32_t *out_cnt = out_cnt_s[tok];
    uint32_t(*col_max)[64] = col_max_s[tok];
    uint32_t *n_cand = n_cand_s[tok];
    uint16_t(*cand)[KVQ_V_CAND] = cand_s[tok];
    float *red_mx = red_mx_s[tok], *red_mn = red_mn_s[tok];
    uint32_t(*bits)[CW + 1] = bits_s[wave];
    uint32_t *mask = mask_s[tok][wave];
    __shared__ float lut_s[NE];
    const int jb = wave * JW;                    // this wavefront's first channel group (D = 64 W JW)
    // Two tokens of a pair share the dwords of their codes.  TOK = 2: the workgroup has both (or, at either end
    // of the call, one: the other's wavefronts then repeat its work and store nothing).
    const int t_mine = TOK == 1 ? first : 2 * first + tok - (int)(n0 & 1);
    const bool valid = TOK == 1 || (t_mine >= 0 && t_mine < T);
    const int t = valid ? t_mine : (tok == 0 ? t_mine + 1 : t_mine - 1);
    const int64_t n = n0 + t;
    const uint16_t *x16 = v_new + (int64_t)t * D + lane;
    const uint32_t base = v_ptr[n0] + (uint32_t)t * 2u * (uint32_t)k_side;
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    const uint32_t K = (uint32_t)k_side;

    uint16_t xc[JW];                             // this lane's elements, kept in registers
    auto load = [&] {
#pragma unroll
        for (int i = 0; i < JW; ++i) xc[i] = x16[64 * (jb + i)];
    };
    if (TOK == 1) load();                        // (a lone token is latency; in bulk the registers are better free)
    KvqParamsView pv = kvq_params_view(params, D);
    const KvqCoder<NE> coder(pv.hdr->thr_v, pv.hdr->lut_v);
    stage_lut<NE>(lut_s, pv.hdr->lut_v);         // (visible after the barrier that follows the ranges)
    if (ttid < 64) {
        col_max[0][ttid] = 0u;
        col_max[1][ttid] = 0u;
        if (ttid < 2) n_cand[ttid] = 0u;
    }
    // the wavefronts' packing areas, cleared here and filled after the barrier that follows the ranges
    for (int e = threadIdx.x; e < W * JW * (CW + 1); e += TOK * NTW) (&bits_s[0][0][0])[e] = 0;
    if (lane <= CW) mask[lane] = 0;
    __syncthreads();
    if (TOK == 2) load();
    uint32_t top = 0, bot = 0;                   // bit i: channel 64 (jb + i) + lane is an upper / lower outlier
    static_assert(JW <= 32, "one mask bit per element of a lane");
    uint32_t kc[JW];                             // the elements' order-preserving keys
    uint32_t kmax = 0, kmin = 0xffffu;           // this lane's extremes
#pragma unroll
    for (int i = 0; i < JW; ++i) {
        const uint32_t key = order_key(xc[i]);
        kc[i] = key;
        kmax = key > kmax ? key : kmax;
        kmin = key < kmin ? key : kmin;
    }
    if (K > 0) {
        // Bounds of the thresholds.  The K-th largest of the 64 columns' largest keys is a lower bound of the
        // token's K-th largest key, since that many elements are at least as large; likewise for the smallest.
        // One wavefront finds each, two key bits at a time, with ballots.  With more outliers per side
        // than KVQ_V_BOUNDED the bounds let more keys pass than a list holds (64 columns: 64 ln(64 / (64 - K)) are
        // expected, 107 for K = 52): none are taken, every key goes to the histograms.
        uint32_t tau_top, tau_bot, need_top, need_bot, n_eq_top, n_eq_bot;
        if constexpr (W == 1) {                  // one wavefront has them all
            uint32_t inv[JW];
#pragma unroll
            for (int i = 0; i < JW; ++i) inv[i] = 0xffffu - kc[i];
            wave_threshold<JW>(kc, kmax, K, tau_top, need_top, n_eq_top);
            wave_threshold<JW>(inv, 0xffffu - kmin, K, tau_bot, need_bot, n_eq_bot);
            tau_bot = 0xffffu - tau_bot;
        } else {
        atomicMax(&col_max[0][lane], kmax);
        atomicMax(&col_max[1][lane], 0xffffu - kmin);
        __syncthreads();
        uint32_t m_top = 0, m_bot = 0xffffu;
        if (K <= KVQ_V_BOUNDED) {
            if (wave < 2) {                      // a wavefront a side
                const uint32_t c[1] = {col_max[wave][lane]}, x = wave_rank<1, 8>(c, K);
                if (lane == 0) bound_s[tok][wave] = x;
            }
            __syncthreads();
            m_top = bound_s[tok][0];
            m_bot = 0xffffu - bound_s[tok][1];
        }
        // The few keys on and beyond the bounds (24 a side are expected of 4096 for K = 20) are collected,
        // in any order, and the thresholds are found among them.
        uint32_t which = 0;                      // bit i: element i is a candidate
#pragma unroll
        for (int i = 0; i < JW; ++i) which |= (K <= KVQ_V_BOUNDED && (kc[i] >= m_top || kc[i] <= m_bot)) ? (1u << i) : 0u;
        // With many equal keys every key would be read again and counted on two words of LDS (64 tokens of 4096 equal
        // channels: 40 us): from the third round on a wavefront stops when a list is full, since the lists are of no
        // use then (see below).  (Not from what the additions return: waiting for it costs one token 0.4 us.)
        int round = 0;
        while (__ballot(which != 0u) != 0ull) {  // (most lanes have none, hardly any more than two)
            if (++round > 2 && (__hip_atomic_load(&n_cand[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > KVQ_V_CAND ||
                                __hip_atomic_load(&n_cand[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > KVQ_V_CAND))
                break;
            if (which != 0u) {
                const int i = __ffs((int)which) - 1;
                which &= which - 1u;
                // (a dynamic index: few elements are looked through, many read again)
                uint32_t key = kc[0];
                if constexpr (JW <= 8) {
#pragma unroll
                    for (int j = 1; j < JW; ++j) key = i == j ? kc[j] : key;
                } else {
                    key = order_key(x16[64 * (jb + i)]);
                }
                if (key >= m_top) {
                    const uint32_t at = atomicAdd(&n_cand[0], 1u);
                    if (at < KVQ_V_CAND) cand[0][at] = (uint16_t)key;
                }
                if (key <= m_bot) {
                    const uint32_t at = atomicAdd(&n_cand[1], 1u);
                    if (at < KVQ_V_CAND) cand[1][at] = (uint16_t)(0xffffu - key);
                }
            }
        }
        __syncthreads();
        const uint32_t nt = n_cand[0], nb = n_cand[1];
        bool few = K <= KVQ_V_BOUNDED && nt <= KVQ_V_CAND && nb <= KVQ_V_CAND;
        if (TOK == 2) {                          // (barriers below: both tokens take the same way)
            const uint32_t *other = n_cand_s[TOK - 1 - tok];
            few = few && other[0] <= KVQ_V_CAND && other[1] <= KVQ_V_CAND;
        }
        if (few) {
            // K-th largest candidate of either list, which has at least K entries; its keys lie between the bound and the largest, + 1
            // from the bound, so that an absent entry is below all
            if (wave < 2) {
                const uint32_t n = wave ? nb : nt, from = bound_s[tok][wave];
                constexpr int R = KVQ_V_CAND / 64;
                uint32_t v[R], most = 0;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const uint32_t e = (uint32_t)lane + 64u * r;
                    v[r] = e < n ? cand[wave][e] - from + 1u : 0u;
                    most = v[r] > most ? v[r] : most;
                }
                const int steps = (33 - __builtin_clz(wave_magnitude(most))) / 2;
                const uint32_t x = wave_rank<R, 9>(v, K, steps);
                auto at_least = [&](uint32_t y) {
                    uint32_t c = 0;
#pragma unroll
                    for (int r = 0; r < R; ++r) c += (uint32_t)__popcll(__ballot(v[r] >= y));
                    return c;
                };
                const uint32_t beyond = at_least(x + 1u), reached = at_least(x);
                if (lane == 0) {
                    found_s[tok][wave][0] = x - 1u + from;
                    found_s[tok][wave][1] = beyond;
                    found_s[tok][wave][2] = reached - beyond;
                }
            }
            __syncthreads();
            tau_top = found_s[tok][0][0];
            tau_bot = 0xffffu - found_s[tok][1][0];
            need_top = K - found_s[tok][0][1];
            need_bot = K - found_s[tok][1][1];
            n_eq_top = found_s[tok][0][2];
            n_eq_bot = found_s[tok][1][2];
        } else {
            // Many equal keys, or more outliers per side than the bounds serve: radix selection on histograms,
            // of the keys that passed.  Counts are exact from the bounds outwards, which is all the searches read.
            for (int i = ttid; i < 768; i += NTW) hist[i] = 0;
            __syncthreads();
            // more than half of this wavefront's first keys in one bin (asked of two lanes)
            const uint32_t b0 = kc[0] >> 8;
            const bool tied = __popcll(__ballot(b0 == (uint32_t)__builtin_amdgcn_readlane((int)b0, 0))) > 32 ||
                              __popcll(__ballot(b0 == (uint32_t)__builtin_amdgcn_readlane((int)b0, 32))) > 32;
            auto count_high = [&](auto t) {
#pragma unroll
                for (int i = 0; i < JW; ++i) {
                    const uint32_t key = kc[i];
                    hist_count(hist, key >= m_top || key <= m_bot, key >> 8, lane, decltype(t)::value);
                }
            };
            if (tied) count_high(std::true_type{});
            else count_high(std::false_type{});
            __syncthreads();
            uint32_t bin_top, above_top, in_top, bin_bot, below_bot, in_bot;
            wave_find_bin<true>(hist, K, lane, bin_top, above_top, in_top);
            wave_find_bin<false>(hist, K, lane, bin_bot, below_bot, in_bot);
            auto count_low = [&](auto t) {
#pragma unroll
                for (int i = 0; i < JW; ++i) {
                    const uint32_t key = kc[i];
                    hist_count(hist + 256, (key >> 8) == bin_top && key >= m_top, key & 255u, lane, decltype(t)::value);
                    hist_count(hist + 512, (key >> 8) == bin_bot && key <= m_bot, key & 255u, lane, decltype(t)::value);
                }
            };
            if (tied) count_low(std::true_type{});
            else count_low(std::false_type{});
            __syncthreads();
            uint32_t lo_top, above_in, lo_bot, below_in;
            wave_find_bin<true>(hist + 256, K - above_top, lane, lo_top, above_in, n_eq_top);
            wave_find_bin<false>(hist + 512, K - below_bot, lane, lo_bot, below_in, n_eq_bot);
            tau_top = (bin_top << 8) | lo_top;
            tau_bot = (bin_bot << 8) | lo_bot;
            need_top = K - (above_top + above_in);
            need_bot = K - (below_bot + below_in);
        }
        }
        const bool same = tau_top == tau_bot;
        // ranks of equal keys are only needed when some but not all of them are taken (the same in all of a
        // token's wavefronts; with two tokens the barrier is reached whatever either needs)
        const bool ranked = same || need_top != n_eq_top || need_bot != n_eq_bot;
        uint32_t run_top = 0, run_bot = 0;       // equal keys before this wavefront's channels, then running
        if (ranked) {
            uint32_t ct = 0, cb = 0;
#pragma unroll
            for (int i = 0; i < JW; ++i) {
                const uint32_t key = kc[i];
                ct += (uint32_t)__popcll(__ballot(key == tau_top));
                cb += (uint32_t)__popcll(__ballot(key == tau_bot));
            }
            if (lane == 0) { eq_cnt[wave][0] = ct; eq_cnt[wave][1] = cb; }
            if (TOK == 1) __syncthreads();
        }
        if (TOK == 2) __syncthreads();
        if (ranked)
            for (int w = 0; w < wave; ++w) { run_top += eq_cnt[w][0]; run_bot += eq_cnt[w][1]; }
#pragma unroll
        for (int i = 0; i < JW; ++i) {
            const uint32_t key = kc[i];
            const bool eq_t = key == tau_top, eq_b = key == tau_bot;
            bool is_top, is_bot;
            if (ranked) {
                const unsigned long long bt = __ballot(eq_t), bb = __ballot(eq_b);
                const uint32_t rt = run_top + (uint32_t)__popcll(bt & lt_mask);
                const uint32_t rb = run_bot + (uint32_t)__popcll(bb & lt_mask);
                run_top += (uint32_t)__popcll(bt);
                run_bot += (uint32_t)__popcll(bb);
                is_top = key > tau_top || (eq_t && rt < need_top);
                // thresholds coincide: the lower outliers take the equal keys that follow the upper ones'
                is_bot = !is_top && (key < tau_bot ||
                                     (eq_b && (same ? (rb >= need_top && rb < need_top + need_bot) : rb < need_bot)));
            } else {
                is_top = key >= tau_top;
                is_bot = key <= tau_bot;
            }
            top |= (uint32_t)is_top << i;
            bot |= (uint32_t)is_bot << i;
        }
    }
    // range of the remaining elements, and this wavefront's number of outliers
    float mx = -INFINITY, mn = INFINITY;
    const uint32_t outl = top | bot;
#pragma unroll
    for (int i = 0; i < JW; ++i)
        if (!((outl >> i) & 1u)) { const float x = kvq_h2f(xc[i]); mx = fmaxf(mx, x); mn = fminf(mn, x); }
    uint32_t n_out = 0;
    if constexpr (JW <= 8) {                     // (no trip through LDS: latency is what a call of few tokens is made of)
#pragma unroll
        for (int i = 0; i < JW; ++i) n_out += (uint32_t)__popcll(__ballot((outl >> i) & 1u));
        mx = kvq_wave_max(mx);
        mn = -kvq_wave_max(-mn);
    } else {
        n_out = (uint32_t)__popc(outl);
        for (int o = 32; o > 0; o >>= 1) {
            mx = fmaxf(mx, __shfl_xor(mx, o));
            mn = fminf(mn, __shfl_xor(mn, o));
            n_out += __shfl_xor(n_out, o);
        }
    }
    if (lane == 0) { red_mx[wave] = mx; red_mn[wave] = mn; out_cnt[wave] = n_out; }
    __syncthreads();
    mx = red_mx[0]; mn = red_mn[0];
#pragma unroll
    for (int w = 1; w < W; ++w) { mx = fmaxf(mx, red_mx[w]); mn = fminf(mn, red_mn[w]); }
    uint32_t running = 0;                        // outliers before this wavefront's channels, then running
    for (int w = 0; w < wave; ++w) running += out_cnt[w];
    const float sum = mx + mn, dif = mx - mn;
    uint16_t zb = kvq_f2h_rn(sum * 0.5f), sb = kvq_f2h_rn(dif * 0.5f);
    float zf = kvq_h2f(zb), sf = kvq_h2f(sb);
    if (sf == 0.0f) { sf = 1.0f; sb = 0x3c00u; }
    const float rinv = __fdiv_rn(1.0f, sf);
    if (ttid == 0 && valid) { v_sz[n * 2 + 0] = sb; v_sz[n * 2 + 1] = zb; }

    const int parity = (int)(n & 1);
    bool overflow = false;
    auto encode = [&](auto calm) {
#pragma unroll
        for (int i = 0; i < JW; ++i) {
            const int j = jb + i;
            const float x = kvq_h2f(xc[i]);
            const float diff = x - zf;
            const float xn = diff * rinv;
            const int code = decltype(calm)::value ? coder.count(xn) : coder(xn);
            const bool is_out = (outl >> i) & 1u;
            const unsigned long long b = __ballot(is_out);
            if (is_out && valid) {
                const uint64_t pos = (uint64_t)base + running + (uint32_t)__popcll(b & lt_mask);
                if (pos < (uint64_t)cap_nnz)
                    vsp.put(pos, (uint16_t)(64 * j + lane), kvq_f2h_rn(x - __builtin_fmaf(sf, lut_s[code], zf)));
                else overflow = true;
            }
            running += (uint32_t)__popcll(b);
            // the chunk of (head j >> 1, half j & 1): this token's bits of 64 fields, gathered in the
            // wavefront's own LDS slice
            if (valid) stream_or(bits[i], lane * 2 * BITS + parity * BITS, (uint32_t)code, BITS);
        }
    };
    // (normalising is monotone: a lane whose extremes are in the coder's range has all its elements there)
    const float d_hi = key_value(kmax) - zf, d_lo = key_value(kmin) - zf;
    if (__ballot(coder.far(d_hi * rinv) || coder.far(d_lo * rinv)) == 0ull) encode(std::true_type{});
    else encode(std::false_type{});
    if (TOK == 2) {
        __syncthreads();                         // both tokens' codes are in the packing areas
        if (T - 2 * first + (int)(n0 & 1) >= 2 && 2 * first >= (int)(n0 & 1)) {
            // both tokens of the pair: whole dwords
            for (int e = threadIdx.x; e < W * JW * CW; e += TOK * NTW) {
                const int j = e / CW, d = e - j * CW;
                *(uint32_t *)(v_codes + kvq_v_piece0(BITS, cap, n >> 1, j >> 1, j & 1) + (d >> 2) * 1024 + (d & 3) * 4) =
                    bits_s[j / JW][j % JW][d];
            }
        }
    }
    if (TOK == 1 || (valid && (2 * first < (int)(n0 & 1) || T - 2 * first + (int)(n0 & 1) < 2))) {
        stream_or(mask, lane * 2 * BITS + parity * BITS, (uint32_t)(NE - 1), BITS);
        // LDS operations of one wavefront execute in order; the fence keeps the compiler from moving the
        // reads below above the atomics
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (int e = lane; e < JW * CW; e += 64) {
            const int i = e / CW, d = e - i * CW, j = jb + i;
            const int64_t off = kvq_v_piece0(BITS, cap, n >> 1, j >> 1, j & 1) + (d >> 2) * 1024 + (d & 3) * 4;
            uint32_t *p = (uint32_t *)(v_codes + off);
            // the partner token of the pair owns the other bits of this dword: clear this token's bits, then
            // set them, with two atomics that return nothing (as in v_quant_token)
            __hip_atomic_fetch_and(p, ~mask[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_or(p, bits[i][d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (ttid == 0 && valid) {
        uint64_t p = (uint64_t)base + 2u * (uint32_t)k_side;
        if (p > (uint64_t)cap_nnz) { p = (uint64_t)cap_nnz; overflow = true; }
        v_ptr[n + 1] = (uint32_t)p;
    }
    if (overflow) atomicExch(d_status, (int32_t)KVQ_ERR_NNZ_OVERFLOW);
}

template <int BITS, int JW, int W, int TOK, class SP>
__global__ __launch_bounds__(64 * W * TOK) void kvq_v_quant4(const void *__restrict__ params, int D, int64_t cap,
                                                          int64_t n0, int T, int k_side,
                                                          const uint16_t *__restrict__ v_new,
                                                          uint8_t *__restrict__ v_codes, uint16_t *__restrict__ v_sz,
                                                          uint32_t *__restrict__ v_ptr, const SP vsp, int64_t cap_nnz,
                                                          int32_t *d_status, const KeyCount keys)
{
    if (TOK == 2 && (int)blockIdx.x < keys.wgs) {
        const int t = (int)blockIdx.x * (W * TOK) + (int)(threadIdx.x >> 6);
        if (t < T) k_count_token<true>(params, D, keys.k_new, keys.cnt, t);
        return;
    }
    v_quant_token4<BITS, JW, W, TOK>(params, D, cap, n0, k_side, v_new, v_codes, v_sz, v_ptr, vsp, cap_nnz, d_status,
                                     (int)blockIdx.x - (TOK == 2 ? keys.wgs : 0), T);
}

// HW = 0: the body for any number of heads.
template <int BITS, int HW, int W, class SP>
__global__ __launch_bounds__(64 * W) void kvq_k_quant(const void *__restrict__ params, int D, int64_t cap, int64_t n0,
                                                      const uint16_t *__restrict__ k_new, uint8_t *__restrict__ k_codes,
                                                      uint32_t *__restrict__ k_ptr, const SP ksp, int64_t cap_nnz, int single,
                                                      int32_t *d_status)
{
    if constexpr (HW == 0)
        k_quant_token<BITS, 64 * W>(params, D, cap, n0, k_new, k_codes, k_ptr, ksp, cap_nnz, single, d_status, (int)blockIdx.x);
    else
        k_quant_token_w<BITS, HW, W>(params, D, cap, n0, k_new, k_codes, k_ptr, ksp, cap_nnz, single, d_status, (int)blockIdx.x);
}

template <int BITS, int NT, class SP>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT == 256 ? 8 : 4)))
void kvq_v_quant(const void *__restrict__ params, int D, int64_t cap, int64_t n0,
                                                  int k_side, const uint16_t *__restrict__ v_new,
                                                  uint8_t *__restrict__ v_codes, uint16_t *__restrict__ v_sz,
                                                  uint32_t *__restrict__ v_ptr, const SP vsp, int64_t cap_nnz, int32_t *d_status)
{
    v_quant_token<BITS, NT>(params, D, cap, n0, k_side, v_new, v_codes, v_sz, v_ptr, vsp, cap_nnz, d_status,
                            (int)blockIdx.x);
}

// Keys and Values of the same tokens in one launch: even workgroups take a token's Keys, odd ones its
// Values (a single-token append is pure latency, and the two do not depend on each other).
template <class SP>
struct KvAppendArgs {
    const void *params;
    int D, k_side, single;
    int64_t cap, n0_k, n0_v, cap_nnz_k, cap_nnz_v;
    const uint16_t *k_new, *v_new;
    uint8_t *k_codes, *v_codes;
    uint16_t *v_sz;
    uint32_t *k_ptr, *v_ptr;
    SP ksp, vsp;
    int32_t *d_status;
};
// NT threads.  VJ, VW: the Values take v_quant_token4 with VJ elements per lane of VW wavefronts, VJ = 0: the routine
// for any width.  One instantiation per width: static LDS of several widths would add up.
template <int BITS, int NT, int VJ, int VW, class SP>
__global__ __launch_bounds__(NT) void kvq_kv_quant(const KvAppendArgs<SP> a)
{
    const int t = (int)(blockIdx.x >> 1);
    if ((blockIdx.x & 1) == 0) {
        // a workgroup's wavefronts share out the heads (see the launch rule of kvq_quantize_append_k)
        constexpr int W = NT / 64;
#define KW(HW)                                                                                                  \
    k_quant_token_w<BITS, HW, W>(a.params, a.D, a.cap, a.n0_k, a.k_new, a.k_codes, a.k_ptr, a.ksp, a.cap_nnz_k,  \
                                 a.single, a.d_status, t)
        if constexpr (VJ > 0) {
            KW((64 * VJ * VW / KVQ_HEAD_DIM + W - 1) / W);
        } else {
            const int hw = (a.D / KVQ_HEAD_DIM + W - 1) / W;
            if (hw == 1) KW(1);
            else if (hw == 2) KW(2);
            else if (hw == 3) KW(3);
            else if (NT == 256 || hw == 4) KW(4);            // (narrow workgroups have fewer than 16 heads)
            else
                k_quant_token<BITS, NT>(a.params, a.D, a.cap, a.n0_k, a.k_new, a.k_codes, a.k_ptr, a.ksp, a.cap_nnz_k,
                                        a.single, a.d_status, t);
        }
#undef KW
    } else if constexpr (VJ > 0) {
        // wavefronts of the workgroup that the routine does not use end here (a barrier waits only for the
        // wavefronts that have not ended)
        if (threadIdx.x >= 64 * VW) return;
        v_quant_token4<BITS, VJ, VW, 1>(a.params, a.D, a.cap, a.n0_v, a.k_side, a.v_new, a.v_codes, a.v_sz, a.v_ptr,
                                        a.vsp, a.cap_nnz_v, a.d_status, t, 0);
    } else
        v_quant_token<BITS, NT>(a.params, a.D, a.cap, a.n0_v, a.k_side, a.v_new, a.v_codes, a.v_sz, a.v_ptr, a.vsp, a.cap_nnz_v, a.d_status, t);
}

// ---- first launch of a generation step ---------------------------------------------------------
// kvq_decode_step appends one token and then attends over the cache that ends with it.  The append is
// two workgroups of pure latency (12 us), and the attention's first kernel, the sparse Key kernel, needs
// the new token only for the last of its scores: here both run as workgroups of one launch.  Workgroup 0
// quantizes the token's Key (k_quant_token_w on sixteen or eight wavefronts, within the registers of the sparse
// kernel's eight wavefronts per SIMD) and then adds up the sparse part of the token's own scores from
// the entries it has just stored; workgroup 1 quantizes its Value; the others are the sparse Key
// kernel over the tokens that were there before.
struct StepFrontArgs {
    const void *params;
    int D, n_q_heads, k_side;
    int64_t cap, n;                       // n: tokens in the cache before the step
    int64_t cap_nnz_k, cap_nnz_v;
    const uint16_t *k_new, *v_new;
    uint8_t *k_codes, *v_codes;
    uint16_t *v_sz;
    uint32_t *k_ptr, *v_ptr;
    KvqSparseFlat ksp, vsp;
    int32_t *d_status;
    const float *q_rot;
    float scale;
    float *scores;
    int64_t ld, tokens_per_wave;
};

// Sparse part of the scores of token a.n, whose entries the NT threads left in this workgroup
// have just stored: scale * v * (R_n^T q)_c summed per query head, as the sparse kernel does for the
// other tokens (same arithmetic per entry; 64-bit fixed-point sums in LDS).
template <int R, int NT>
__device__ __forceinline__ void qk_sparse_new_token(const StepFrontArgs &a)
{
    extern __shared__ __attribute__((aligned(16))) float sparse_dyn[];
    unsigned long long *S = (unsigned long long *)sparse_dyn;            // [n_q_heads]
    const int tid = threadIdx.x;
    for (int j = tid; j < a.n_q_heads; j += NT) S[j] = 0ull;
    // the workgroup's stores of the token's entries and of its end pointer are complete ...
    __threadfence_block();
    __syncthreads();
    // ... and are read back past the vector cache, which may hold the pointer's line from before
    const uint32_t p0 = __hip_atomic_load(a.k_ptr + a.n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t p1 = __hip_atomic_load(a.k_ptr + a.n + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const KvqParamsView pv = kvq_params_view(a.params, a.D);
    for (uint32_t e = p0 + (uint32_t)tid; e < p1; e += NT) {
        const uint32_t ch = __hip_atomic_load(a.ksp.idx + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const float v = kvq_h2f(__hip_atomic_load(a.ksp.val + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        const uint32_t i = ch & 63u;
        const float rev = rope_rev((float)a.n, pv.hdr->rope_vh[i], pv.hdr->rope_vl[i]);
        const float cs = __builtin_amdgcn_cosf(rev);
        // (R_n^T q)_c = q_c cos + s q_{c^64} sin, s = +1 for the lower channel of the pair, -1 for the upper
        const float sn = __builtin_bit_cast(
            float, __builtin_bit_cast(uint32_t, __builtin_amdgcn_sinf(rev)) ^ ((ch & 64u) << 25));
        const uint32_t cl = ch & 127u, kvh = ch >> 7;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t qh = kvh * R + r, qi = qh * 128u + cl;
            const float qa = a.q_rot[qi] * a.scale, qb = a.q_rot[qi ^ 64u] * a.scale;
            const float qp = qa * cs + qb * sn;
            kvq_lds_add_fixed<0>(&S[qh], v * qp);
        }
    }
    __syncthreads();
    for (int j = tid; j < a.n_q_heads; j += NT) a.scores[(int64_t)j * a.ld + a.n] = kvq_from_fixed_fast<0>(S[j]);
}

// ROOMY: sixteen wavefronts per compute unit instead of 32, for contexts that do not fill more (the append roles are then
// the launch's length: 16 us with their registers spilled at 2048 tokens of 4096 channels with 4-bit codes, 10.4 us without).
// W: wavefronts on the Value token (D = 256 W channels: 16 or 4).  One instantiation per width: the
// Value routine's static LDS arrays of several widths would add up and cost the sparse role a workgroup
// per compute unit.
template <int BITS, int R, int W, bool ROOMY>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(ROOMY ? 4 : 8, ROOMY ? 4 : 8)))
void kvq_step_front(const StepFrontArgs)
{
    // The argument block is read where a role needs it, through a pointer the compiler cannot see
    // through.  Read as a kernel argument it is loaded whole at the kernel's entry, fifty scalar
    // registers that stay alive through all three roles and are spilled into vector-register lanes at
    // once; their reloads (v_readlane) then sit in the sparse role's loops, 25 % more VALU instructions
    // in a role that is bound by them.
#if defined(__HIP_DEVICE_COMPILE__)           // (the host pass only needs the kernel's signature)
    typedef const StepFrontArgs __attribute__((address_space(4))) *ArgsPtr;
    ArgsPtr pa = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();      // the one argument sits at offset 0
    asm volatile("" : "+s"(pa));
    if (blockIdx.x == 0) {
        // wavefronts that a role does not use end here (a barrier waits only for those that have not ended)
        constexpr int KW = W == 16 ? 16 : 8, HW = W == 16 ? 2 : 1;         // 32 or 8 heads
        if (threadIdx.x >= 64 * KW) return;
        const StepFrontArgs a = *pa;
        k_quant_token_w<BITS, HW, KW>(a.params, a.D, a.cap, a.n, a.k_new, a.k_codes, a.k_ptr, a.ksp, a.cap_nnz_k, 1,
                                      a.d_status, 0);
        qk_sparse_new_token<R, 64 * KW>(a);
    } else if (blockIdx.x == 1) {
        if (threadIdx.x >= 64 * W) return;
        const StepFrontArgs a = *pa;
        v_quant_token4<BITS, 4, W, 1>(a.params, a.D, a.cap, a.n, a.k_side, a.v_new, a.v_codes, a.v_sz, a.v_ptr, a.vsp,
                                      a.cap_nnz_v, a.d_status, 0, 1);
    } else {
        const KvqSparseFlat ksp{pa->ksp.idx, pa->ksp.val};
        qk_sparse_body<R, 8, KvqSparseFlat>((int)blockIdx.x - 2, pa->params, pa->D, pa->n_q_heads, pa->n, pa->k_ptr, ksp,
                                            (uint32_t)pa->cap_nnz_k, pa->q_rot, pa->scale, pa->scores, pa->ld,
                                            pa->tokens_per_wave);
    }
#endif
}

}  // namespace

// The first n_sink tokens are also kept as they came (paper Sec. 3.5): copy their rows.
static kvq_status copy_sink_rows(const kvq_cache *cache, uint16_t *sink, const uint16_t *src, int64_t n0, int32_t T,
                                 hipStream_t s)
{
    if (n0 >= cache->n_sink) return KVQ_OK;
    const int64_t rows = (cache->n_sink - n0 < T) ? cache->n_sink - n0 : T;
    const size_t D = (size_t)cache->n_kv_heads * KVQ_HEAD_DIM;
    KVQ_HIP_CHECK(hipMemcpyAsync(sink + n0 * D, src, (size_t)rows * D * 2, hipMemcpyDeviceToDevice, s));
    return KVQ_OK;
}

// Workgroup width of the quantization kernels.  A token's workgroup spends most of its time between
// barriers; 1024 threads finish a token soonest (what a decode step needs), while 256-thread
// workgroups, four to a compute unit and out of step with each other, get more tokens per second out
// of a bulk append.
static bool wide_wg(int D, int T) { return D >= 2048 && T < KVQ_BULK_TOKENS; }

// Widths whose Values stay in registers in calls of a few tokens: D / 1024 for whole multiples of 1024 channels up to
// 8192, spread over four (1024), eight (2048) or sixteen wavefronts with D / 1024 elements per lane; 0 for the others,
// whose tokens v_quant_token selects from in LDS.
static int small_width(int D) { return D % 1024 == 0 && D <= 8192 ? D / 1024 : 0; }
// One to three heads, in bulk four: a wavefront per Value token, D / 64 elements per lane (0: wider).  us per Value append, 256 threads a token with
// the selection in LDS / a wavefront: 4096 tokens of 128 channels, 2 bits 17.2 / 8.0, of 256 18.0 / 8.3, of 384 20.4 / 12.6, of 512 21.5 / 15.3; but 1000
// tokens of 512, 4 bits, 11.4 / 10.7, 100 8.0 / 8.9; the append kernel of a step of one head 6.2 / 4.5.  Three heads in short calls, where the six
// elements a lane make the searches longer than the 256 threads' radix selection (Keys and Values, blocked outlier storage, us): one token, 2 bits
// 6.1 / 6.4, 3 bits 6.6 / 6.8, 4 bits 7.1 / 7.2; 200 tokens 11.2 / 11.6, 11.8 / 12.0, 12.2 / 12.0; 300 tokens 14.2 / 14.0; no outliers, one token 4.1 / 3.0.
static int narrow_width(int bits, int D, int T, int k_side)
{
    if (D == 384 && k_side > 0 && bits < 4 && T < KVQ_KV_SPLIT_TOKENS) return 0;
    return D <= (T >= 2048 ? 512 : 384) ? D / 128 : 0;
}

static kvq_status append_checks(const kvq_cache *cache, const void *src, int32_t T, int64_t n_now)
{
    kvq_status st = kvq_check_cache(cache);
    if (st != KVQ_OK) return st;
    if (!cache->loaded) return KVQ_ERR_NOT_LOADED;
    if (!src || ((uintptr_t)src & 1) || T < 1 || T > KVQ_MAX_APPEND) return KVQ_ERR_INVALID_ARG;
    if (n_now + T > cache->cap_tokens) return KVQ_ERR_CAPACITY;
    return KVQ_OK;
}

// counted: the tokens' outliers have been counted into the workspace on this stream already.
static kvq_status append_k(kvq_cache *cache, const uint16_t *d_k_new, int32_t T, void *stream, bool counted)
{
    kvq_status st = append_checks(cache, d_k_new, T, cache ? cache->n_tokens_k : 0);
    if (st != KVQ_OK) return st;
    const int D = cache->n_kv_heads * KVQ_HEAD_DIM;
    hipStream_t s = (hipStream_t)stream;
    const int single = (T == 1);
    // us, kvq_k_bulk / the kernels below with kvq_ptr_scan before them: 64 tokens of 4096 channels, 3 bits 10.0 / 12.4; 777 12.6 / 17.2; 4096 27.0 / 40.5;
    // of 1024 channels, 4096 13.9 / 16.2; of 5120, 4 bits 47.0 / 56.2; of 8192 56.1 / 85.8.  But where codes are searched for, not counted, which here
    // a lane does one by one (signposts past 1): 4096 tokens of 4096 channels, 3 bits 129 / 49, 777 of 5120, 4 bits, 74 / 31, 64 of 4096 23 / 12.
    const bool bulk = T >= KVQ_VW_SMALL_TOKENS && D % 1024 == 0 && D <= 1024 * KVQ_BULK_MAX_WAVES && ((uintptr_t)d_k_new & 15) == 0 &&
                      cache->workspace_bytes >= ((int64_t)T + 3) / 4 * 16 && !(cache->loaded & KVQ_LOADED_SEARCH_K);
    if (!single) {
        if (!cache->workspace || cache->workspace_bytes < (int64_t)T * 4) return KVQ_ERR_CAPACITY;
        uint32_t *cnt = (uint32_t *)cache->workspace;
        if (!counted) {
            const int grid = (T + KVQ_COUNT_NT / 64 - 1) / (KVQ_COUNT_NT / 64);
            if (bulk) kvq_k_count<true><<<grid, KVQ_COUNT_NT, 0, s>>>(cache->params, D, T, d_k_new, cnt);
            else kvq_k_count<false><<<grid, KVQ_COUNT_NT, 0, s>>>(cache->params, D, T, d_k_new, cnt);
        }
        if (!bulk) kvq_ptr_scan<<<1, 1024, 0, s>>>(cache->k_ptr, cache->n_tokens_k, T, cnt, cache->cap_nnz_k, cache->d_status);
    }
#define LAUNCH_KW(B, HW, W)                                                                                     \
    kvq_k_quant<B, HW, W><<<T, 64 * (W), 0, s>>>(cache->params, D, cache->cap_tokens, cache->n_tokens_k, d_k_new, \
                                                 cache->k_codes, cache->k_ptr, ksp, cache->cap_nnz_k, single,    \
                                                 cache->d_status)
    // From KVQ_WAVE_TOKENS tokens on a wavefront each; below, sixteen wavefronts share out a token's heads (four
    // where there are no more than four heads), up to four each.  Wider models take the body that loops, in bulk with
    // 256 threads, of which a compute unit holds several (3 bits, 72 heads, us with 1024 / 256 threads / a wavefront per
    // token: 256 tokens 25 / 32 / 48, 600 tokens 51 / 39 / 49, 1500 tokens 89 / 50 / 67, 3000 tokens 162 / 77 / 73; 128 heads: 512
    // tokens 54 / 58 / 100, 600 tokens 71 / 61 / 99).
#define LAUNCH_K(B)                                                                                             \
    do {                                                                                                        \
        const int H = cache->n_kv_heads;                                                                        \
        if (T >= (H > 16 ? 2 : 1) * KVQ_WAVE_TOKENS)                                                            \
            kvq_k_quant_wave<B><<<(T + KVQ_KW_NT / 64 - 1) / (KVQ_KW_NT / 64), KVQ_KW_NT, 0, s>>>(               \
                cache->params, D, T, cache->cap_tokens, cache->n_tokens_k, d_k_new, cache->k_codes,              \
                cache->k_ptr, ksp, cache->cap_nnz_k, cache->d_status);                                           \
        else if (H <= 4) LAUNCH_KW(B, 1, 4);                                                                    \
        else if (H <= 16) LAUNCH_KW(B, 1, 16);                                                                  \
        else if (H <= 32) LAUNCH_KW(B, 2, 16);                                                                  \
        else if (H <= 48) LAUNCH_KW(B, 3, 16);                                                                  \
        else if (H <= 64) LAUNCH_KW(B, 4, 16);                                                                  \
        else if (T < KVQ_BULK_TOKENS) LAUNCH_KW(B, 0, 16);                                                      \
        else LAUNCH_KW(B, 0, 4);                                                                                \
    } while (0)
    // one set of kernels per layout of the outlier entries (flat arrays or a list of blocks)
    const auto launch = [&](const auto ksp) {
        if (bulk) kvq_k_bulk_launch(cache, d_k_new, T, (const uint32_t *)cache->workspace, s);
        else if (cache->bits == 2) LAUNCH_K(2);
        else if (cache->bits == 3) LAUNCH_K(3);
        else LAUNCH_K(4);
    };
    if (cache->nnz_block_shift) launch(kvq_blocked_k(cache));
    else launch(kvq_flat_k(cache));
#undef LAUNCH_K
#undef LAUNCH_KW
    KVQ_HIP_CHECK(hipGetLastError());
    st = copy_sink_rows(cache, cache->sink_k, d_k_new, cache->n_tokens_k, T, s);
    if (st != KVQ_OK) return st;
    cache->n_tokens_k += T;
    return KVQ_OK;
}

extern "C" kvq_status kvq_quantize_append_k(kvq_cache *cache, const uint16_t *d_k_new, int32_t T, void *stream)
{
    return append_k(cache, d_k_new, T, stream, false);
}

// k_new: null, or the Keys of the same tokens, whose outliers are to be counted into the workspace by the same launch where
// its kernel does that (*counted).
static kvq_status append_v(kvq_cache *cache, const uint16_t *d_v_new, int32_t T, void *stream, const uint16_t *k_new, bool *counted)
{
    kvq_status st = append_checks(cache, d_v_new, T, cache ? cache->n_tokens_v : 0);
    if (st != KVQ_OK) return st;
    const int D = cache->n_kv_heads * KVQ_HEAD_DIM;
    if (cache->k_side_v < 0 || 2 * (int64_t)cache->k_side_v >= D) return KVQ_ERR_INVALID_ARG;
    if (D > 16384) return KVQ_ERR_UNSUPPORTED;       // the per-token selection keeps the vector in LDS
    hipStream_t s = (hipStream_t)stream;
    const size_t dyn = 3 * (size_t)D;
#define LAUNCH_V4W(B, J, WV, TOK, GRID)                                                                        \
    kvq_v_quant4<B, J, WV, TOK><<<(GRID) + keys.wgs, 64 * (WV) * (TOK), 0, s>>>(                               \
        cache->params, D, cache->cap_tokens, cache->n_tokens_v, T, cache->k_side_v, d_v_new, cache->v_codes,   \
        cache->v_sz, cache->v_ptr, vsp, cache->cap_nnz_v, cache->d_status, keys)
    const int small = T < KVQ_VW_SMALL_TOKENS ? small_width(D) : 0, narrow = narrow_width(cache->bits, D, T, cache->k_side_v);
    const bool in_pairs = !small && (D == 4096 || D == 2048 || D == 1024 || (T >= KVQ_BULK_TOKENS && (D == 5120 || D == 6656 || D == 8192)));
    // The pair kernel, one wavefront per 1024 channels and pair, takes calls of 64 tokens and more, but of one or two wavefronts a pair only
    // longer ones: below, a token of 1024 or 2048 channels is sooner done by four wavefronts (us, four / one or two wavefronts: 1024 channels,
    // 2 bits, 777 tokens 9.1 / 11.3, 1200 11.5 / 11.8, 2048 16.2 / 10.6, 4 bits, 1200 12.3 / 13.4, 2048 17.8 / 12.0; 2048 channels, 777 tokens 11.3 / 11.9
    // and 13.1 / 14.7, 1200 14.5 / 9.9 and 17.3 / 11.5).  More than KVQ_V_BOUNDED outliers a side, other widths and unaligned input keep the
    // other kernels.  So do calls of up to 4 M elements whose codes are searched for, not counted, which here a lane does one by one (signposts past 1,
    // us, four wavefronts a token / this one: 64 tokens of 4096 channels, 3 bits 16.0 / 19.2, 777 20.3 / 19.9, 4 bits 18.6 / 24.0, 25.1 / 26.4, 4096 75.6 /
    // 71.1, 1000 of 2048 16.2 / 26.9, 4096 of 1024 31.2 / 34.0; but 2 bits, 64 of 4096 13.1 / 11.1; of 5120, 4 bits, 24.4 / 26.2, 1500 44.7 / 39.2).
    const bool searched = (cache->loaded & KVQ_LOADED_SEARCH_V) && cache->bits > 2;
    const bool pair = !small && D % 1024 == 0 && D <= 1024 * KVQ_BULK_MAX_WAVES && cache->k_side_v <= (int)KVQ_V_BOUNDED &&
                      ((uintptr_t)d_v_new & 15) == 0 && T >= (D == 1024 ? 1500 : D == 2048 ? 1000 : KVQ_VW_SMALL_TOKENS) &&
                      !(searched && in_pairs && D <= 4096 && (int64_t)T * D <= (4 << 20));
    KeyCount keys = {0, nullptr, nullptr};
    // Counting on the way saves a launch and its latency (32 heads, blocked storage, 2048 tokens, us with a launch of its own / on the way: 2 bits 34.1 /
    // 31.1, 4 bits 42.6 / 39.4; 4096 tokens 49.3 / 46.7, 65.0 / 62.4; 16 heads 33.7 / 33.5, 42.2 / 43.2), except in the kernel of four wavefronts a token from
    // 2048 tokens of 2048 or 4096 channels on with blocked outlier storage, which has no vector time to spare.
    const bool busy = !pair && cache->nnz_block_shift && T >= 2048 && (D == 2048 || D == 4096);
    const bool count = k_new != nullptr && (in_pairs || pair) && !busy;
    if (counted) *counted = count;
    const int wg_waves = pair ? D / 1024 : 2 * KVQ_VW_WAVES;
    if (count) keys = {(T + wg_waves - 1) / wg_waves, k_new, (uint32_t *)cache->workspace};
    // a workgroup per pair of tokens (the two that share dwords), the first and the last perhaps with one token
    const unsigned pairs = (unsigned)(((cache->n_tokens_v + T - 1) >> 1) - (cache->n_tokens_v >> 1) + 1);
#define LAUNCH_V4(B, J) LAUNCH_V4W(B, J, KVQ_VW_WAVES, 2, pairs)
#define LAUNCH_V(B)                                                                                             \
    do {                                                                                                        \
        if (narrow == 1) LAUNCH_V4W(B, 2, 1, 1, T);                                                             \
        else if (narrow == 2) LAUNCH_V4W(B, 4, 1, 1, T);                                                        \
        else if (narrow == 3) LAUNCH_V4W(B, 6, 1, 1, T);                                                        \
        else if (narrow == 4) LAUNCH_V4W(B, 8, 1, 1, T);                                                        \
        else if (small == 1) LAUNCH_V4W(B, 4, 4, 1, T);                                                              \
        else if (small == 2) LAUNCH_V4W(B, 4, 8, 1, T);                                                         \
        else if (small == 3) LAUNCH_V4W(B, 3, 16, 1, T);                                                        \
        else if (small == 4) LAUNCH_V4W(B, 4, 16, 1, T);                                                        \
        else if (small == 5) LAUNCH_V4W(B, 5, 16, 1, T);                                                        \
        else if (small == 6) LAUNCH_V4W(B, 6, 16, 1, T);                                                        \
        else if (small == 7) LAUNCH_V4W(B, 7, 16, 1, T);                                                        \
        else if (small == 8) LAUNCH_V4W(B, 8, 16, 1, T);                                                        \
        else if (D == 4096) LAUNCH_V4(B, 16);                                                                   \
        else if (D == 2048) LAUNCH_V4(B, 8);                                                                    \
        else if (D == 1024) LAUNCH_V4(B, 4);                                                                    \
        else if (D == 5120 && T >= KVQ_BULK_TOKENS) LAUNCH_V4(B, 20);                                           \
        else if (D == 6656 && T >= KVQ_BULK_TOKENS) LAUNCH_V4(B, 26);                                           \
        else if (D == 8192 && T >= KVQ_BULK_TOKENS) LAUNCH_V4(B, 32);                                           \
        else if (wide_wg(D, T))                                                                                 \
            kvq_v_quant<B, 1024><<<T, 1024, dyn, s>>>(cache->params, D, cache->cap_tokens, cache->n_tokens_v,    \
                                                      cache->k_side_v, d_v_new, cache->v_codes, cache->v_sz,     \
                                                      cache->v_ptr, vsp,                                         \
                                                      cache->cap_nnz_v, cache->d_status);                        \
        else                                                                                                    \
            kvq_v_quant<B, 256><<<T, 256, dyn, s>>>(cache->params, D, cache->cap_tokens, cache->n_tokens_v,      \
                                                    cache->k_side_v, d_v_new, cache->v_codes, cache->v_sz,       \
                                                    cache->v_ptr, vsp, cache->cap_nnz_v,                        \
                                                    cache->d_status);                                            \
    } while (0)
    const auto launch = [&](const auto vsp) {
        if (pair) kvq_v_pair_launch(cache, d_v_new, T, pairs, keys.wgs, keys.k_new, keys.cnt, s);
        else if (cache->bits == 2) LAUNCH_V(2);
        else if (cache->bits == 3) LAUNCH_V(3);
        else LAUNCH_V(4);
    };
    if (cache->nnz_block_shift) launch(kvq_blocked_v(cache));
    else launch(kvq_flat_v(cache));
#undef LAUNCH_V
#undef LAUNCH_V4
#undef LAUNCH_V4W
    KVQ_HIP_CHECK(hipGetLastError());
    st = copy_sink_rows(cache, cache->sink_v, d_v_new, cache->n_tokens_v, T, s);
    if (st != KVQ_OK) return st;
    cache->n_tokens_v += T;
    return KVQ_OK;
}

extern "C" kvq_status kvq_quantize_append_v(kvq_cache *cache, const uint16_t *d_v_new, int32_t T, void *stream)
{
    return append_v(cache, d_v_new, T, stream, nullptr, nullptr);
}

extern "C" kvq_status kvq_quantize_append_kv(kvq_cache *cache, const uint16_t *d_k_new, const uint16_t *d_v_new,
                                             int32_t T, void *stream)
{
    kvq_status st = append_checks(cache, d_k_new, T, cache ? cache->n_tokens_k : 0);
    if (st != KVQ_OK) return st;
    st = append_checks(cache, d_v_new, T, cache->n_tokens_v);
    if (st != KVQ_OK) return st;
    const int D = cache->n_kv_heads * KVQ_HEAD_DIM;
    if (cache->k_side_v < 0 || 2 * (int64_t)cache->k_side_v >= D) return KVQ_ERR_INVALID_ARG;
    if (D > 16384) return KVQ_ERR_UNSUPPORTED;       // the per-token Value selection keeps the vector in LDS
    const bool searched = (cache->loaded & (KVQ_LOADED_SEARCH_K | KVQ_LOADED_SEARCH_V)) != 0;
    // (what the bulk kernels take; 4096 channels have a Value kernel for pairs of tokens besides)
    const bool bulk = D % 1024 == 0 && D <= 1024 * KVQ_BULK_MAX_WAVES && !searched &&
                      (D == 4096 || (cache->k_side_v <= (int)KVQ_V_BOUNDED && (((uintptr_t)d_k_new | (uintptr_t)d_v_new) & 15) == 0));
    const int split = !bulk || (D <= 2048 && cache->bits > 2) ? KVQ_KV_SPLIT_TOKENS : D <= 2048 ? KVQ_KV_SPLIT_NARROW : KVQ_KV_SPLIT_BULK;
    if (T >= split) {
        // Such an append fills the GPU with either kernel alone.  From 129 tokens on, two workgroups of 1024 threads per token are more than the
        // compute units hold at once, and the bulk kernels are the faster ones, but hardly of one or two wavefronts a token (us in one launch / in turn: 129
        // tokens, 4 bits, 24 heads 22.6 / 15.7, 40 heads 26.8 / 17.6, 16 heads 12.9 / 14.3, 8 heads 10.9 / 11.8; 165 tokens 13.6 / 14.5, 11.4 / 12.0, 255 14.6 /
        // 14.7, 11.7 / 12.1; blocked storage, 200 tokens, 3 bits 13.8 / 14.5, 12.0 / 12.4, but 2 bits 13.5 / 13.1, 11.7 / 11.3; 64 heads 33 / 18; 100 tokens,
        // 40 heads 18.0 / 19.1).  Other widths, 255 tokens, 4 bits: 52 heads 68 / 48.  What the bulk kernels do not take, 40 heads, 130
        // tokens, 2 bits: 60 outliers a side 23.7 / 32.1, unaligned input 31.4 / 41.0, but 32 heads 21.7 / 18.5, 28.4 / 19.0; codes that are searched for, 150 tokens, 4 bits 31.9 / 34.6.
        // Every check of both calls has passed above.
        if (!cache->workspace || cache->workspace_bytes < (int64_t)T * 4) return KVQ_ERR_CAPACITY;
        // Values first: their kernel counts the Keys' outliers on the way (see KeyCount).
        bool counted = false;
        st = append_v(cache, d_v_new, T, stream, d_k_new, &counted);
        if (st != KVQ_OK) return st;
        return append_k(cache, d_k_new, T, stream, counted);
    }
    hipStream_t s = (hipStream_t)stream;
    const int single = (T == 1);
    if (!single) {
        if (!cache->workspace || cache->workspace_bytes < (int64_t)T * 4) return KVQ_ERR_CAPACITY;
        uint32_t *cnt = (uint32_t *)cache->workspace;
        kvq_k_count<false><<<(T + KVQ_COUNT_NT / 64 - 1) / (KVQ_COUNT_NT / 64), KVQ_COUNT_NT, 0, s>>>(cache->params, D, T, d_k_new, cnt);
        kvq_ptr_scan<<<1, 1024, 0, s>>>(cache->k_ptr, cache->n_tokens_k, T, cnt, cache->cap_nnz_k, cache->d_status);
    }
    const size_t dyn = 3 * (size_t)D;
    const int narrow = narrow_width(cache->bits, D, T, cache->k_side_v);
    static_assert(KVQ_KV_SPLIT_TOKENS <= KVQ_BULK_TOKENS, "workgroups are wide for every D >= 2048 here");
#define LAUNCH_KVW(B, NT, VJ, VW) kvq_kv_quant<B, NT, VJ, VW><<<2 * T, NT, (VJ) > 0 ? 0 : dyn, s>>>(a)
#define LAUNCH_KV(B)                                                                     \
    do {                                                                                 \
        switch (narrow ? -narrow : small_width(D)) {                                     \
        case -1: LAUNCH_KVW(B, 256, 2, 1); break;                                        \
        case -2: LAUNCH_KVW(B, 256, 4, 1); break;                                        \
        case -3: LAUNCH_KVW(B, 256, 6, 1); break;                                        \
        case 1: LAUNCH_KVW(B, 256, 4, 4); break;                                         \
        case 2: LAUNCH_KVW(B, 1024, 4, 8); break;                                        \
        case 3: LAUNCH_KVW(B, 1024, 3, 16); break;                                       \
        case 4: LAUNCH_KVW(B, 1024, 4, 16); break;                                       \
        case 5: LAUNCH_KVW(B, 1024, 5, 16); break;                                       \
        case 6: LAUNCH_KVW(B, 1024, 6, 16); break;                                       \
        case 7: LAUNCH_KVW(B, 1024, 7, 16); break;                                       \
        case 8: LAUNCH_KVW(B, 1024, 8, 16); break;                                       \
        default:                                                                         \
            if (wide_wg(D, T)) LAUNCH_KVW(B, 1024, 0, 0);                                \
            else LAUNCH_KVW(B, 256, 0, 0);                                               \
        }                                                                                \
    } while (0)
    const auto launch = [&](const auto ksp, const auto vsp) {
        KvAppendArgs<std::remove_cv_t<decltype(ksp)>> a;
        a.params = cache->params; a.D = D; a.k_side = cache->k_side_v; a.single = single;
        a.cap = cache->cap_tokens; a.n0_k = cache->n_tokens_k; a.n0_v = cache->n_tokens_v;
        a.cap_nnz_k = cache->cap_nnz_k; a.cap_nnz_v = cache->cap_nnz_v;
        a.k_new = d_k_new; a.v_new = d_v_new;
        a.k_codes = cache->k_codes; a.v_codes = cache->v_codes; a.v_sz = cache->v_sz;
        a.k_ptr = cache->k_ptr; a.v_ptr = cache->v_ptr;
        a.ksp = ksp; a.vsp = vsp;
        a.d_status = cache->d_status;
        if (cache->bits == 2) LAUNCH_KV(2);
        else if (cache->bits == 3) LAUNCH_KV(3);
        else LAUNCH_KV(4);
    };
    if (cache->nnz_block_shift) launch(kvq_blocked_k(cache), kvq_blocked_v(cache));
    else launch(kvq_flat_k(cache), kvq_flat_v(cache));
#undef LAUNCH_KV
#undef LAUNCH_KVW
    KVQ_HIP_CHECK(hipGetLastError());
    st = copy_sink_rows(cache, cache->sink_k, d_k_new, cache->n_tokens_k, T, s);
    if (st != KVQ_OK) return st;
    st = copy_sink_rows(cache, cache->sink_v, d_v_new, cache->n_tokens_v, T, s);
    if (st != KVQ_OK) return st;
    cache->n_tokens_k += T;
    cache->n_tokens_v += T;
    return KVQ_OK;
}


template <int BITS, int R, int W, bool ROOMY>
static kvq_status step_front_launch_brw(kvq_cache *cache, StepFrontArgs &a, hipStream_t s, bool *done, bool dry)
{
    // static LDS of the kernel (the append bodies' arrays) comes on top of the sparse role's dynamic LDS
    static const int static_lds = [] {
        hipFuncAttributes fa;
        if (hipFuncGetAttributes(&fa, (const void *)kvq_step_front<BITS, R, W, ROOMY>) != hipSuccess) return -1;
        return (int)fa.sharedSizeBytes;
    }();
    static const hipError_t lds_attr = hipFuncSetAttribute((const void *)kvq_step_front<BITS, R, W, ROOMY>,
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, 147456 - 16384);
    if (static_lds < 0 || static_lds > 16384) return KVQ_OK;             // *done stays false
    KVQ_HIP_CHECK(lds_attr);
    QkSparsePlan plan;
    if (!qk_sparse_plan(cache->n_q_heads, a.n, 8, (size_t)static_lds, ROOMY ? 1 : 2, plan) || plan.waves != 16) return KVQ_OK;
    if (plan.lds < (size_t)cache->n_q_heads * 8) return KVQ_OK;
    a.tokens_per_wave = plan.tokens_per_wave;
    if (dry) {                                    // the caller only asks whether this launch applies
        *done = true;
        return KVQ_OK;
    }
    kvq_status st = copy_sink_rows(cache, cache->sink_k, a.k_new, a.n, 1, s);
    if (st != KVQ_OK) return st;
    st = copy_sink_rows(cache, cache->sink_v, a.v_new, a.n, 1, s);
    if (st != KVQ_OK) return st;
    kvq_step_front<BITS, R, W, ROOMY><<<plan.grid + 2, 1024, plan.lds, s>>>(a);
    KVQ_HIP_CHECK(hipGetLastError());
    cache->n_tokens_k += 1;
    cache->n_tokens_v += 1;
    *done = true;
    return KVQ_OK;
}

template <int BITS, int R>
static kvq_status step_front_launch_br(kvq_cache *cache, StepFrontArgs &a, hipStream_t s, bool *done, bool dry)
{
    // 4096 channels: up to twelve tokens per wavefront of one workgroup per compute unit, the launch with the registers
    // that the append roles of 4-bit codes want: with two workgroups per unit they spill 44.  us per step with one / two, 32 heads,
    // 4 bits: 300 tokens 33.6 / 37.8, 8192 36.8 / 41.2, 16384 43.0 / 47.9, 32768 63.9 / 67.0, 48000 89.8 / 91.2, 52000 94.6 / 97.2, 65536 109.4 /
    // 105.3.  2- and 3-bit codes spill nothing in either; one workgroup per unit then has half as many runs to start and end, which
    // gains 1 to 3 % up to 24000 tokens and 1 % or less either way from there: 2 bits, 8192 tokens 31.8 / 32.4, 24000 43.5 / 44.8, 32768 49.6 /
    // 49.2, 48000 64.1 / 63.7, 65536 78.4 / 73.5; 3 bits, 8192 31.7 / 32.4, 24000 48.1 / 49.5, 32768 54.5 / 54.1, 48000 71.6 / 71.8, 65536 87.4 / 81.9.
    // (1024 channels spill nothing: 8 heads, 4 bits, 16000 tokens 32.6 / 30.7.)
    if (a.D == 4096)
        return a.n <= 12 * 16 * (int64_t)kvq_cu_count() ? step_front_launch_brw<BITS, R, 16, true>(cache, a, s, done, dry)
                                                        : step_front_launch_brw<BITS, R, 16, false>(cache, a, s, done, dry);
    return step_front_launch_brw<BITS, R, 4, false>(cache, a, s, done, dry);
}

template <int BITS>
static kvq_status step_front_launch_b(kvq_cache *cache, StepFrontArgs &a, hipStream_t s, bool *done, bool dry)
{
    switch (cache->n_q_heads / cache->n_kv_heads) {
    case 1: return step_front_launch_br<BITS, 1>(cache, a, s, done, dry);
    case 2: return step_front_launch_br<BITS, 2>(cache, a, s, done, dry);
    case 4: return step_front_launch_br<BITS, 4>(cache, a, s, done, dry);
    case 8: return step_front_launch_br<BITS, 8>(cache, a, s, done, dry);
    default: return KVQ_OK;
    }
}

static kvq_status step_front(kvq_cache *cache, const uint16_t *d_k_new, const uint16_t *d_v_new,
                             const float *d_q_rot, float scale, float *d_scores, int64_t ld_scores, hipStream_t s,
                             bool *done, bool dry)
{
    *done = false;
    kvq_status st = append_checks(cache, d_k_new, 1, cache ? cache->n_tokens_k : 0);
    if (st != KVQ_OK) return st;
    st = append_checks(cache, d_v_new, 1, cache->n_tokens_v);
    if (st != KVQ_OK) return st;
    const int D = cache->n_kv_heads * KVQ_HEAD_DIM;
    if (cache->k_side_v < 0 || 2 * (int64_t)cache->k_side_v >= D) return KVQ_ERR_INVALID_ARG;
    // shapes this launch covers; every other one takes the two calls
    if (D != 1024 && D != 4096) return KVQ_OK;
    if (cache->nnz_block_shift || (cache->loaded & 2) || cache->n_tokens_k != cache->n_tokens_v) return KVQ_OK;
    if (cache->cap_nnz_k >= ((int64_t)1 << 31)) return KVQ_OK;
    const int64_t per_token = cache->cap_nnz_k / (cache->cap_tokens > 0 ? cache->cap_tokens : 1);
    if (per_token < 16 && cache->n_q_heads <= 32) return KVQ_OK;         // the sparse kernel would take 32-token sub-ranges
    StepFrontArgs a;
    a.params = cache->params; a.D = D; a.n_q_heads = cache->n_q_heads; a.k_side = cache->k_side_v;
    a.cap = cache->cap_tokens; a.n = cache->n_tokens_k;
    a.cap_nnz_k = cache->cap_nnz_k; a.cap_nnz_v = cache->cap_nnz_v;
    a.k_new = d_k_new; a.v_new = d_v_new;
    a.k_codes = cache->k_codes; a.v_codes = cache->v_codes; a.v_sz = cache->v_sz;
    a.k_ptr = cache->k_ptr; a.v_ptr = cache->v_ptr;
    a.ksp = kvq_flat_k(cache); a.vsp = kvq_flat_v(cache);
    a.d_status = cache->d_status;
    a.q_rot = d_q_rot; a.scale = scale; a.scores = d_scores; a.ld = ld_scores; a.tokens_per_wave = 1;
    if (cache->bits == 2) return step_front_launch_b<2>(cache, a, s, done, dry);
    if (cache->bits == 3) return step_front_launch_b<3>(cache, a, s, done, dry);
    return step_front_launch_b<4>(cache, a, s, done, dry);
}

kvq_status kvq_step_front_launch(kvq_cache *cache, const uint16_t *d_k_new, const uint16_t *d_v_new,
                                 const float *d_q_rot, float scale, float *d_scores, int64_t ld_scores, hipStream_t s,
                                 bool *done)
{
    return step_front(cache, d_k_new, d_v_new, d_q_rot, scale, d_scores, ld_scores, s, done, false);
}

extern "C" int32_t kvq_decode_step_launches(const kvq_cache *cache)
{
    if (!cache) return -1;
    kvq_cache view = *cache;                     // a dry run: nothing is launched, nothing advances
    bool front = false;
    static const uint16_t dummy[2] = {0, 0};     // the checks only look at alignment
    if (step_front(&view, dummy, dummy, nullptr, 0.f, nullptr, 0, nullptr, &front, true) != KVQ_OK) return -1;
    const int sink = cache->n_sink > 0 ? 1 : 0;
    // the two calls: append, sparse Key (unless the thresholds admit no outlier), dense Key, sparse Value,
    // dense Value, reduction
    const int two_calls = (cache->loaded & 2) ? 5 : 6;
    view.n_tokens_v = cache->n_tokens_v + 1;     // what the Value half of the step covers
    return (front ? 5 : two_calls) + sink - (kvq_pv_is_one_launch(&view) ? 1 : 0);
}
