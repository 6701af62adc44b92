// Attention output against the quantized Value cache (paper Sec. 3.1 per-token Values, App. "Kernel
// Implementation Details"): dense look-up-table mat-vec plus the sparse outlier mat-vec, merged into
// one result.
//
// Design (gfx950).  out[q][c] = sum_n p[q][n] (s_n lut[code_{n,c}] + z_n) + sparse.  The storage format
// keeps the codes of two consecutive tokens of one channel side by side in a 2b-bit field, so one LDS
// gather of the fp16 pair (lut[a], lut[b]) from a layer-wide table gives two consecutive elements of a
// matrix-core operand; the weights w = p*s, split in three fp16 parts, are the other operand (kvq_pv_dense).
// The zero-point term sum_n p z_n is a per-head scalar.  Sparse outliers are handled by a balanced kernel
// (lanes = outlier entries, fixed-point LDS accumulators), in one launch with the dense one where neither fills the chip
// (kvq_pv_both); all partial results, and the fp16 rows of
// attention-sink tokens (paper Sec. 3.5) if any, are summed in a fixed order by a final small kernel.
#include "kvq_common.hpp"
#include <math.h>
#include <type_traits>

namespace {

constexpr int PV_TILE = 64;                // tokens per tile of the dense kernel (32 token pairs)
constexpr int PV_CHAIN = 16;               // tiles whose products one accumulator takes up
constexpr size_t PV_BOTH_LDS = 160 * 1024; // most LDS of a workgroup
constexpr int PV_MIN_TILES = 8;            // tiles a workgroup should at least have: half of its wavefronts busy

// The sparse kernel's wavefronts take consecutive runs of `units` times `unit` tokens (8 or 16), the first `longer` of them
// one unit more.
struct PvsRuns {
    int unit, units, longer;
};

struct PvPlan {
    int slabs;              // workgroups per head group of the dense kernel (tiles are split evenly among them)
    int tiles;              // tiles of PV_TILE tokens
    int sslabs;             // workgroups of the sparse kernel
    int swaves;             // its wavefronts per workgroup
    int64_t tokens_per_swave;   // a multiple of 8
    size_t slds;            // its dynamic LDS bytes
};

constexpr int PVS_TW = 16;                // tokens per sub-range of a sparse-kernel wavefront
// row length of the staged probabilities: one token's outliers read the same column of many rows,
// and an odd row length spreads that column over all LDS banks
constexpr int PVS_ROW = PVS_TW + 1;
constexpr int PVS_U = 8;                  // 64-entry batches in flight per wavefront
constexpr int PVS_MAX_SLABS = 512;

__host__ __device__ constexpr int pvs_wave_lds_floats(int n_q_heads)
{
    return n_q_heads * PVS_ROW;                          // the sub-range's probabilities
}

// Query heads of one KV head that a wavefront of the dense kernel takes together (they share the codes): a group of
// several saves gathers and reads per tile and costs start and end of the kernel (maxima, sums over lanes and
// wavefronts, one head after the other), so it pays once a wavefront has tiles enough.  Counted in tiles per
// wavefront of the whole GPU with one head each: one head up to 1, two up to 3, four up to 12.  Measured, kvq_pv_matvec,
// us with groups of 8 / 4 / 2 / 1 heads: 32 heads on 4, 2-bit, 1000 tokens (1/8 tile) 17.6 / 14.6 / 14.1 / 14.2, 12000
// (1.5) 18.6 / 16.0 / 15.4 / 15.6; 3-bit, 24000 (2.9) 19.4 / 18.6 / 18.6 / 20.8, 48000 (5.9) 24.7 / 24.8 / 26.3 / 31.4, 131000
// (16) 32.7 / 33.3 / 39.7 / 54.7; 64 on 8, 4-bit, 6000 (1.5) 31.5 / 28.8 / 28.8 / 29.8, 24000 (5.9) 38.6 / 37.6 / 39.5 / 44.6,
// 131000 (32) 68.8 / 71.8 / 84.1 / 114.5.
inline int pv_group(int64_t L, int n_q_heads, int r)
{
    const int64_t tiles = n_q_heads * ((L + PV_TILE - 1) / PV_TILE), waves = 16 * (int64_t)kvq_cu_count();
    int rg = tiles <= waves ? 1 : tiles <= 3 * waves ? 2 : tiles <= 12 * waves ? 4 : 8;
    while (r % rg) rg >>= 1;
    return rg;
}

inline PvPlan pv_plan(int64_t L, int n_q_heads, int rg)
{
    PvPlan p;
    const int64_t tiles = (L + PV_TILE - 1) / PV_TILE;
    // one workgroup per compute unit (its table and staging take most of the LDS), none with fewer than
    // PV_MIN_TILES tiles
    int64_t want = (int64_t)kvq_cu_count() / (n_q_heads / rg);
    if (want > (tiles + PV_MIN_TILES - 1) / PV_MIN_TILES) want = (tiles + PV_MIN_TILES - 1) / PV_MIN_TILES;
    if (want > 512) want = 512;
    if (want < 1) want = 1;
    p.tiles = (int)tiles;
    p.slabs = (int)want;
    // sparse kernel: LDS holds Hq*128 64-bit accumulators shared by the workgroup plus a private slice
    // per wavefront (two workgroups of 12 wavefronts per CU when they fit in 77 KiB each); the launch
    // fills the chip once (256 CUs, 160 KiB of LDS and 24 wavefronts each, at most PVS_MAX_SLABS
    // workgroups) and every wavefront gets the same number of tokens (a multiple of 8)
    int waves = 12;
    const size_t per_wave = (size_t)pvs_wave_lds_floats(n_q_heads) * 4;
    const size_t shared = (size_t)n_q_heads * (1024 + 8);      // accumulators + per-head score maxima (8 bytes each: alignment)
    while (waves > 1 && shared + waves * per_wave > 78848) waves -= (waves > 4) ? 4 : waves / 2;
    p.swaves = waves;
    p.slds = shared + waves * per_wave;
    int wgs_per_cu = (int)(163840 / p.slds);
    if (wgs_per_cu * waves > 24) wgs_per_cu = 24 / waves;      // six wavefronts per SIMD (register budget)
    if (wgs_per_cu < 1) wgs_per_cu = 1;
    int64_t max_wgs = (int64_t)kvq_cu_count() * wgs_per_cu;
    if (max_wgs > PVS_MAX_SLABS) max_wgs = PVS_MAX_SLABS;
    const int64_t resident = max_wgs * waves;
    int64_t tpw = (L + resident - 1) / resident;
    tpw = (tpw + 7) & ~(int64_t)7;
    if (tpw < 8) tpw = 8;
    const int64_t n_waves = (L + tpw - 1) / tpw;
    p.tokens_per_swave = tpw;
    p.sslabs = (int)((n_waves + waves - 1) / waves);
    if (p.sslabs < 1) p.sslabs = 1;
    return p;
}

// Bits before the point (without the sign) of the sparse sums of a workgroup of `tokens` tokens, 64-bit words.  The fused
// call's weights are 1 at most: enough for the largest fp16 residual (65504, and a margin for weights whose exponent is
// rounded) in every token.  A caller's own weights: 23 in a launch of its own, of `own` tokens a workgroup; as much per
// token in a larger workgroup.
inline int pv_whole_bits(int64_t tokens, int64_t own, bool fused)
{
    int bits = 23;
    while ((fused ? tokens * 66000 >> bits : tokens > own << (bits - 23)) && bits < 62) ++bits;
    return bits;
}

// Plan of the one launch for both kernels.  The compute units are dealt out so that either kind takes as long, by its work in
// us per 131072 tokens on the whole chip: sparse 2 (pointers), 0.12 per query head (scores staged) and 0.08 + 0.11 per query
// head of the KV head for an outlier, times 1.22 (eight-head groups: 2) because its wavefronts have 16 (8) beside them on a
// compute unit here and up to 24 in their own kernel; dense, per head group, 1.0, 1.4 or 1.5 (2, 3, 4 bits) and 0.2 more for
// every head of a group beyond the first.  Sparse runs differ by one unit at most, so that the time has no steps along L:
// with every run rounded up to the longest, 131073 tokens of 32 heads took 6 % more sparse time than 131072.
//
// One launch is taken where it is estimated to end sooner than two, by work of the same form with the constants that separate
// some 3500 measured shapes best (1 to 40 KV heads, 1 to 8 query heads each, 2 to 4 bits, 0.1 and 1 % outliers, 2048 to 524288 tokens:
// kvq_pv_matvec and kvq_attention_decode with either form forced); a second launch and the first and last round trips of a
// kernel cost 9.26 us.  36 of the shapes are more than 2 % slower in the form taken (8.5 % at most, mostly 16 KV heads with 0.1 %
// outliers), where runs rounded up and constants from sixty shapes left 101 (15 %).  Both sides grow with L in proportion, so a shape
// has one context from which on there are two launches.
// kvq_attention_decode, us, two launches / one: 3-bit, 32 heads, 2048 tokens 28.3 / 24.2, 16383 43.2 / 37.3, 65536 86.1 / 82.1, 82500 102.1 /
// 103.1, 110000 127.0 / 125.6, 131072 137.3 / 135.7 (in a step 132.8 / 129.0), 150000 (two from 189000 on) 159.6 / 162.8; 4-bit 32768 70.3 / 61.0; 32 on 8, 2-bit
// 131100 102.3 / 96.3, 262144 136.8 / 135.4, 524288 (two) 241.9 / 246.1; 64 on 8, 3-bit, 98500 163 / 133, 524288 529 / 475; 32 on 4, 4-bit, 57000 66.4 / 58.4,
// 262144 (two) 136 / 149; 40 heads, 3-bit, 50000 112.0 / 108.7 (five calls), 90000 (two) 126.5 / 131.5; one head, 4096 26.3 / 18.7, 524288 55.7 / 50.2.
//
// Below 2048 tokens two launches would be the slower ones too (32 heads, 300 tokens 26.2 / 23.3, 1600 27.0 / 24.0; one head 21.6 / 18.2, 22.3 /
// 18.8): they stay because kvq_decode_step_launches states five or six launches there, and its results are part of the interface.
struct PvBoth {
    int n_sparse, slabs;               // sparse workgroups (of the dense one's width), dense ones per head group
    PvsRuns runs;                      // of the sparse ones
    int64_t most_tokens;               // of one of these workgroups
    size_t lds;
};
inline bool pv_both(const kvq_cache *c, int rg, size_t dense_lds, PvBoth &p)
{
    const int Hq = c->n_q_heads, r = Hq / c->n_kv_heads;
    const int64_t L = c->n_tokens_v;
    if (c->cap_nnz_v >= ((int64_t)1 << 31) || L < 2048) return false;
    const int waves = rg == 8 ? 8 : 16, cus = kvq_cu_count(), groups = Hq / rg;
    const size_t sparse_lds = (size_t)Hq * (1024 + 8) + (size_t)waves * pvs_wave_lds_floats(Hq) * 4;
    p.lds = sparse_lds > dense_lds ? sparse_lds : dense_lds;
    if (p.lds > PV_BOTH_LDS) return false;
    const double sparse = (2.0 + 0.12 * Hq + 2.0 * c->k_side_v * (0.08 + 0.11 * r)) * (rg == 8 ? 2.0 : 1.22);
    const double dense = groups * ((c->bits == 2 ? 1.0 : c->bits == 3 ? 1.4 : 1.5) + 0.2 * (rg - 1));
    auto slowest = [&](int slabs) {                        // of the two kinds
        const int left = cus - slabs * groups;
        const double d = dense * cus / (slabs * groups), s = left < 1 ? 1e30 : sparse * cus / left;
        return s > d ? s : d;
    };
    int slabs = (int)(cus * dense / ((dense + sparse) * groups));
    slabs = slabs < 1 ? 1 : slabs;
    if (slowest(slabs + 1) < slowest(slabs)) ++slabs;
    const int left = cus - slabs * groups;
    if (left < 1) return false;
    const int64_t wavefronts = (int64_t)left * waves;
    // (whole sub-ranges, so that the scores of one start on 64 bytes; half ones where that leaves wavefronts without)
    const int unit = L > 64 * wavefronts ? PVS_TW : PVS_TW / 2;
    const int64_t units = (L + unit - 1) / unit;
    p.n_sparse = (int)(units < wavefronts ? (units + waves - 1) / waves : left);
    const int64_t runs = (int64_t)p.n_sparse * waves;
    p.runs = {unit, (int)(units / runs), (int)(units % runs)};
    p.most_tokens = (int64_t)unit * waves * (p.runs.units + (p.runs.longer > 0));
    const int64_t few = ((L + PV_TILE - 1) / PV_TILE + PV_MIN_TILES - 1) / PV_MIN_TILES;
    p.slabs = slabs > few ? (int)few : slabs;
    if (p.n_sparse > PVS_MAX_SLABS || p.slabs > 512) return false;
    const PvPlan two = pv_plan(L, Hq, rg);
    const int own = two.swaves * (int)(PV_BOTH_LDS / two.slds);         // sparse wavefronts on a compute unit in their own kernel
    const double x = (double)L / 131072.0;
    const double sw = 1.45 + 0.0627 * Hq + 2.0 * c->k_side_v * (0.0713 + 0.151 * r);
    const double dw = groups * ((c->bits == 2 ? 1.18 : c->bits == 3 ? 1.76 : 1.34) + 0.182 * (rg - 1));
    const double s_one = sw * (rg == 8 ? 1.35 : 1.23) * cus / left, d_one = dw * cus / (slabs * groups);
    const double s_two = own < 24 ? sw * sqrt(24.0 / own) : sw;
    const int64_t per_group = cus / groups;
    const double d_two = per_group > 0 ? dw * cus / (double)(per_group * groups) : dw;
    // (eight tokens per wavefront at least: short contexts leave compute units over, and the estimate is beside the point)
    return units <= wavefronts || (s_one > d_one ? s_one : d_one) * x <= (s_two + d_two) * x + 9.26;
}

template <int FBITS>
__device__ inline uint32_t pv_field_off(const uint32_t *W, int i, uint32_t lane_off)
{
    // (field value * 128) | lane_off : entry e of the replicated table sits at byte e * 128 + lane_off
    const int bit = i * FBITS, wi = bit >> 5, sh = bit & 31;
    constexpr uint32_t M = ((1u << FBITS) - 1u) << 7;
    uint32_t x;
    if (sh + FBITS <= 32) {
        if (sh >= 7) x = W[wi] >> (sh - 7);
        else x = W[wi] << (7 - sh);
    } else {
        x = __builtin_amdgcn_alignbit(W[wi + 1], W[wi], sh - 7);   // straddling fields start at bit >= 26
    }
    return kvq_and_or(x, M, lane_off);
}

// Dense part: a matrix product on the matrix cores.  A wavefront owns one group of RG query heads that share
// a KV head and takes tiles of 64 tokens.  The right operand of v_mfma_f32_16x16x32_f16 is signposts: column
// n of a step stands for channel 8 n + t (t = 0..7: eight steps cover the KV head's 128 channels), its 32
// rows for 32 tokens, and a lane's eight values are four fields of the storage format as the table returns
// them, (lut[a], lut[b]) of a token pair: fp16 numbers, exact.  The left operand is weights w = p s: row
// 4 h + i holds part i of head h's weights: w = w_0 + 2^-12 w_1 + 2^-24 w_2 under a power-of-two scale per
// wavefront and head that keeps the largest weight below 2^15 (at 2^8 when it is set; lowered, with an exact
// rescaling of the sums, when a tile exceeds it).  Each part is the fp16 number nearest to what the ones before it
// leave, raised by 2^12: all 24 bits of an fp32 weight are held down to 2^-33 of the largest one, and a smaller one to
// 2^-57 of the largest.  (Parts under one common scale end at 2^-24: a weight 2^-20 of the largest, beside an
// attention sink, keeps 13 bits.)  Products are exact and sums fp32, rounded once per instruction (32 tokens); rows
// i = 3 are not used.  A row's sum runs over PV_CHAIN tiles and is then added to the wavefront's (sum[]): at a
// million tokens a wavefront has 8192, and the error against 64 bits on random codes and weights is 1.4e-7 of the
// result instead of 2.8e-7 with one running sum (added every 4 tiles 1.4e-7 too, and 0.5 % slower at 131072 tokens;
// every 16: no difference there or at a million, 56.1 -> 56.4 us for a step of 16384).
//
// Per field a lane spends two instructions (cut the field out, form the table address) and one LDS gather
// (2-bit codes: per pair of fields, whose byte indexes a table of both), whatever RG: the multiply-adds, 2 RG
// instructions per field before, are off the vector ALUs.  What the layout costs is a transposition: a chunk is
// loaded 16 bytes per lane (512 contiguous bytes per half and piece), left in LDS in [pair][128 channels] order (row
// length 32 BITS + 16 bytes) and read back as the lane's four pairs; the next tile's codes are requested as soon as
// the current ones have left their registers.  Bank conflicts: none to speak of with 4-bit codes (0.05 of 109 M LDS
// cycles), 14 % of the LDS cycles with 3-bit codes, 34 % with 2-bit ones.  Weights are computed once per (head, token), one token per lane.
//
// Bound: HBM (5.5 TB/s of loads alone on 131072 tokens of 32 heads, 6.6 TB/s on a million), with VALU and LDS
// about 60 % busy each on 3-bit codes.  Measured against one lane per token pair with fp32 multiply-adds (four
// or two heads sharing a field at most): 524288 tokens, 2-bit, 32 heads on 8: 153 -> 53 us; 33001 tokens, 4-bit,
// 32 on 8: 20.0 -> 13.5 us; one head per KV head: 16384 tokens, 4-bit, 16.0 -> 12 us, 131072 tokens, 3-bit, 50-54 ->
// 47-50 us, a million, 4-bit: HBM-bound before and after (340-400 us).
//
// grid = (slabs, head groups); the wavefronts of a workgroup take its tiles in turn and add their sums
// through LDS.  Writes partial[slab][q][128], zpart[slab][q] and (with statistics) lpart[slab][q].
constexpr float PV_PART_UP = 4096.f, PV_PART_DOWN = 1.f / 4096.f;
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));

template <int BITS, int RG>
struct PvCfg {
    static constexpr int NT = RG == 8 ? 512 : 1024;                 // eight heads: twice the sums, half the wavefronts
    static constexpr int WAVES = NT / 64;
    static constexpr int SETS = (RG + 3) / 4;                       // left operands of 16 rows
    static constexpr int FG = BITS == 2 ? 2 : 1;                    // fields per gather: two 4-bit fields are one byte
    // table of signpost pairs: an entry for every value of FG fields, in copies side by side, one for each bank
    // that a lane's gather may start in.  Rows of 256 bytes (4-bit codes, where they fit): the address of a
    // gather is then two bytes, the field and the lane's place, and one byte permute forms it
    static constexpr bool BYTES = BITS == 4 && RG <= 2;
    static constexpr int ROW = BYTES ? 256 : 128;
    static constexpr int TAB = (1 << (2 * BITS * FG)) * ROW;
    static constexpr int PAIR = 32 * BITS + 16;                     // staged codes of a token pair
    static constexpr int WROW = 2 * PV_TILE + 16;                   // a row of weight parts
    static constexpr int WAVE = (PV_TILE / 2) * PAIR + 3 * RG * WROW;
    static constexpr int LDS = TAB + WAVES * WAVE;
};

template <int BITS, int RG>
__device__ __forceinline__ void pv_dense_body(
    uint8_t *lds, const int slab, const int n_slabs, const int group, const void *__restrict__ params, int D, int n_kv_heads, int n_q_heads, int64_t cap, int64_t L,
    const uint8_t *__restrict__ v_codes, const uint16_t *__restrict__ v_sz, const float *__restrict__ probs, int64_t ld,
    float *__restrict__ partial, float *__restrict__ zpart, int n_tiles, int n_sink,
    const float *__restrict__ stat_slots, int n_stat, float *__restrict__ lpart)
{
    // workgroup `slab` of the n_slabs that share the tiles of head group `group`; lds: C::LDS bytes.
    // tokens below n_sink are attention-sink tokens kept in fp16: their quantized form gets weight 0
    // here and the reduce kernel adds their fp16 rows.
    // stat_slots != null: `probs` holds raw scores x; a wavefront takes the maximum m of each of its
    // heads' n_stat slots once, weights every token by exp(x - m) as it loads its score, and the workgroup
    // also writes the sum of these weights to lpart[slab][q] (the reduce kernel divides by their total)
    using C = PvCfg<BITS, RG>;
    constexpr int WAVES = C::WAVES, SETS = C::SETS;
    static_assert(C::LDS >= WAVES * RG * 130 * 4, "the workgroup's sums reuse the array");
    const KvqParamsView pv = kvq_params_view(params, D);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q0 = group * RG;                                 // first query head of the group
    const int kvh = q0 / (n_q_heads / n_kv_heads);
    const int tile1 = (int)(((int64_t)(slab + 1) * n_tiles) / n_slabs);
    int tile = (int)(((int64_t)slab * n_tiles) / n_slabs) + wave;

    // the tile's loads: lane = token for scores and (scale, zero-point), lane = (half, pair) for the codes
    uint4 cw[BITS];
    float xs[RG];
    uint32_t szw = 0;
    const int64_t plane = (cap >> 1) * 16 * BITS;                   // bytes between the two halves of a KV head
    auto request = [&](int t) {
        const int64_t m = (int64_t)t * (PV_TILE / 2) + (lane & 31);
        const uint8_t *p = v_codes + kvq_v_piece0(BITS, cap, m, kvh, 0) + (lane >> 5) * plane;
#pragma unroll
        for (int j = 0; j < BITS; ++j) cw[j] = kvq_load_stream16(p + j * 1024);
        // (loaded whatever the conditions below say, from an index that exists: a load inside a
        // conditional block is followed by a wait for every load in flight)
        int64_t n = (int64_t)t * PV_TILE + lane;
        n = n < L ? n : L - 1;
        szw = *(const uint32_t *)(v_sz + 2 * n);
#pragma unroll
        for (int h = 0; h < RG; ++h) xs[h] = probs[(int64_t)(q0 + h) * ld + n];
    };
    if (tile < tile1) request(tile);

    float m2[RG], lacc[RG], zacc[RG], scale[RG];
    int expo[RG];                                                   // scale = 2^expo; 0: no tile seen yet
#pragma unroll
    for (int h = 0; h < RG; ++h) { m2[h] = 0.f; lacc[h] = 0.f; zacc[h] = 0.f; scale[h] = 0.f; expo[h] = 0; }
    if (stat_slots) {
        float m[RG];                                                // (the heads' loads are in flight together)
#pragma unroll
        for (int h = 0; h < RG; ++h) m[h] = KVQ_STAT_FLOOR;
        for (int i0 = 0; i0 < n_stat; i0 += 64) {
            const int i = i0 + lane < n_stat ? i0 + lane : n_stat - 1;      // a repeated slot does not change a maximum
#pragma unroll
            for (int h = 0; h < RG; ++h) m[h] = __builtin_fmaxf(m[h], stat_slots[(int64_t)(q0 + h) * KVQ_STAT_SLOTS + i]);
        }
#pragma unroll
        for (int h = 0; h < RG; ++h) m2[h] = kvq_wave_max(m[h]) * KVQ_LOG2E;
    }
    for (int e = tid; e < C::TAB / 4; e += C::NT) {
        const int f = C::FG == 1 ? e / (C::ROW / 4) : ((e >> 5) >> (4 * (e & 1))) & 15;     // field that dword e stands for
        ((half2_t *)lds)[e] = half2_t{(half_t)pv.hdr->lut_v[f & ((1 << BITS) - 1)], (half_t)pv.hdr->lut_v[f >> BITS]};
    }
    __syncthreads();

    const uint32_t lane_off = (uint32_t)(lane & (C::ROW / (4 * C::FG) - 1)) * 4 * C::FG;
    uint8_t *mine = lds + C::TAB + wave * C::WAVE;                  // staged codes, then rows of weight parts
    uint8_t *wrows = mine + (PV_TILE / 2) * C::PAIR;
    const int col = lane & 15, kg = lane >> 4;                      // column / row of an operand, group of 8 tokens
    // where this lane reads its operands: row 4 h + i of a left operand is part i of head h (rows without a
    // meaning read some other row: what they give ends up in sums that nobody reads)
    const uint8_t *arow[SETS];
#pragma unroll
    for (int q = 0; q < SETS; ++q) {
        int h = 4 * q + (col >> 2);
        h = h < RG ? h : RG - 1;
        arow[q] = wrows + (3 * h + ((col & 3) < 3 ? (col & 3) : 2)) * C::WROW + kg * 16;
    }
    // 8 fields = 2 BITS bytes at 2 BITS col; for 3 bits the two dwords around them
    const uint8_t *brow = mine + kg * 4 * C::PAIR + (BITS == 3 ? (col >> 1) * 12 + (col & 1) * 4 : 2 * BITS * col);
    const uint32_t bshift = (uint32_t)(col & 1) * 16;
    float4_t acc[SETS][8];
    float sum[SETS][8];                                             // head 4 q + kg, channel 8 col + t, scaled
#pragma unroll
    for (int q = 0; q < SETS; ++q)
#pragma unroll
        for (int t = 0; t < 8; ++t) { acc[q][t] = float4_t{0.f, 0.f, 0.f, 0.f}; sum[q][t] = 0.f; }
    auto collect = [&] {                                            // the three parts of the weights meet
#pragma unroll
        for (int q = 0; q < SETS; ++q)
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float small = __builtin_fmaf(acc[q][t][2], PV_PART_DOWN, acc[q][t][1]);
                sum[q][t] += __builtin_fmaf(small, PV_PART_DOWN, acc[q][t][0]);
                acc[q][t] = float4_t{0.f, 0.f, 0.f, 0.f};
            }
    };

    for (int chain = 0; tile < tile1; tile += WAVES) {
        if (chain++ == PV_CHAIN) { collect(); chain = 1; }
        const int64_t n = (int64_t)tile * PV_TILE + lane;
        const bool ok = n < L && n >= n_sink;
        const float s = kvq_h2f((uint16_t)(szw & 0xFFFFu)), z = kvq_h2f((uint16_t)(szw >> 16));
        float w[RG], top = 0.f;
#pragma unroll
        for (int h = 0; h < RG; ++h) {
            float p = xs[h];
            if (stat_slots) p = kvq_stat_weight(p, m2[h]);
            p = ok ? p : 0.f;
            lacc[h] += p;
            zacc[h] = __builtin_fmaf(p, z, zacc[h]);
            w[h] = p * s;
            top = __builtin_fmaxf(top, __builtin_fabsf(w[h] * scale[h]));
        }
        // the first tile, or a weight beyond the range of its head's scale (rare: weights have to grow by
        // 2^6 over all that came before): set the scales anew
        if (scale[0] == 0.f || __ballot(!(top < 32768.f)) != 0ull) {
            float ratio[RG];
#pragma unroll
            for (int h = 0; h < RG; ++h) {
                const float m = kvq_wave_max(__builtin_fabsf(w[h]));
                ratio[h] = 1.f;
                if (scale[h] == 0.f || !(m * scale[h] < 32768.f)) {
                    int e = m > 0.f ? 9 - __builtin_amdgcn_frexp_expf(m) : 120;       // m * 2^e in [2^8, 2^9)
                    e = e > 120 ? 120 : e < -120 ? -120 : e;
                    ratio[h] = scale[h] == 0.f ? 0.f : __builtin_ldexpf(1.f, e - expo[h]);
                    scale[h] = __builtin_ldexpf(1.f, e);
                    expo[h] = e;
                }
            }
#pragma unroll
            for (int q = 0; q < SETS; ++q) {
                float r = 1.f;                                      // sums of head h sit in the lanes of group h
#pragma unroll
                for (int h = 0; h < 4 && 4 * q + h < RG; ++h) r = kg == h ? ratio[4 * q + h] : r;
#pragma unroll
                for (int t = 0; t < 8; ++t) { acc[q][t] *= r; sum[q][t] *= r; }
            }
        }
#pragma unroll
        for (int h = 0; h < RG; ++h) {
            const float ws = w[h] * scale[h];
            const half_t a = (half_t)ws;
            const float r1 = (ws - (float)a) * PV_PART_UP;          // (below 2^15 again, and exact)
            const half_t b = (half_t)r1;
            const half_t c = (half_t)((r1 - (float)b) * PV_PART_UP);
            half_t *row = (half_t *)(wrows + 3 * h * C::WROW) + lane;
            row[0] = a;
            row[C::WROW / 2] = b;
            row[C::WROW] = c;
        }
        uint8_t *to = mine + (lane & 31) * C::PAIR + (lane >> 5) * 16 * BITS;
#pragma unroll
        for (int j = 0; j < BITS; ++j) *(uint4 *)(to + 16 * j) = cw[j];
        if (tile + WAVES < tile1) request(tile + WAVES);
        // (LDS operations of one wavefront execute in order; the fences keep the compiler from reordering them)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < PV_TILE / 32; ++k) {
            half8_t a[SETS];
#pragma unroll
            for (int q = 0; q < SETS; ++q) a[q] = *(const half8_t *)(arow[q] + k * 64);
            uint32_t W[4][2];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t *b = (const uint32_t *)(brow + (16 * k + j) * C::PAIR);
                W[j][0] = b[0];
                W[j][1] = BITS == 2 ? 0u : b[1];
                if (BITS == 3) {
                    W[j][0] = __builtin_amdgcn_alignbit(W[j][1], W[j][0], bshift);
                    W[j][1] >>= bshift;
                }
            }
#pragma unroll
            for (int t = 0; t < 8; t += C::FG) {
                uint32_t g[C::FG][4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint8_t *e;
                    if constexpr (C::BYTES) e = lds + __builtin_amdgcn_perm(W[j][t >> 2], lane_off, 0x0c0c0400u + ((t & 3) << 8));
                    else e = lds + pv_field_off<2 * BITS * C::FG>(W[j], t / C::FG, lane_off);
                    if (C::FG == 1) {
                        g[0][j] = *(const uint32_t *)e;
                    } else {
                        const uint2 v = *(const uint2 *)e;
                        g[0][j] = v.x;
                        g[C::FG - 1][j] = v.y;
                    }
                }
#pragma unroll
                for (int u = 0; u < C::FG; ++u) {
                    const half8_t b = __builtin_bit_cast(half8_t, uint4{g[u][0], g[u][1], g[u][2], g[u][3]});
#pragma unroll
                    for (int q = 0; q < SETS; ++q)
                        acc[q][t + u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[q], b, acc[q][t + u], 0, 0, 0);
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    collect();
    // the workgroup's sums: wavefronts leave theirs in LDS, [wave][head][128 channels, zero-point, weights]
#pragma unroll
    for (int h = 0; h < RG; ++h) {
        for (int o = 32; o > 0; o >>= 1) {
            zacc[h] += __shfl_xor(zacc[h], o);
            lacc[h] += __shfl_xor(lacc[h], o);
        }
    }
    __syncthreads();                      // every wavefront has left the table
    float *sums = (float *)lds + wave * RG * 130;
#pragma unroll
    for (int q = 0; q < SETS; ++q) {
        const int h = 4 * q + kg;
        float inv = 0.f;
#pragma unroll
        for (int i = 0; i < 4 && 4 * q + i < RG; ++i) inv = kg == i ? (scale[4 * q + i] == 0.f ? 0.f : __builtin_ldexpf(1.f, -expo[4 * q + i])) : inv;
        if (h < RG) {
#pragma unroll
            for (int t = 0; t < 8; ++t) sums[h * 130 + 8 * col + t] = sum[q][t] * inv;
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int h = 0; h < RG; ++h) { sums[h * 130 + 128] = zacc[h]; sums[h * 130 + 129] = lacc[h]; }
    }
    __syncthreads();
    for (int i = tid; i < RG * 130; i += C::NT) {
        float v = 0.f;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) v += ((const float *)lds)[k * RG * 130 + i];
        const int h = i / 130, c = i - 130 * h;
        const int64_t o = (int64_t)slab * n_q_heads + q0 + h;
        if (c < 128) partial[o * 128 + c] = v;
        else if (c == 128) zpart[o] = v;
        else if (stat_slots) lpart[o] = v;
    }
}

#define KVQ_PV_DENSE_PARAMS                                                                                              \
    const void *__restrict__ params, int D, int n_kv_heads, int n_q_heads, int64_t cap, int64_t L,                     \
        const uint8_t *__restrict__ v_codes, const uint16_t *__restrict__ v_sz, const float *__restrict__ probs,       \
        int64_t ld, float *__restrict__ partial, float *__restrict__ zpart, int n_tiles, int n_sink,                   \
        const float *__restrict__ stat_slots, int n_stat, float *__restrict__ lpart
#define KVQ_PV_DENSE_ARGS                                                                                               \
    params, D, n_kv_heads, n_q_heads, cap, L, v_codes, v_sz, probs, ld, partial, zpart, n_tiles, n_sink, stat_slots,    \
        n_stat, lpart
template <int BITS, int RG, bool SPAN = false>
__global__ __launch_bounds__((PvCfg<BITS, RG>::NT)) void kvq_pv_dense(KVQ_PV_DENSE_PARAMS, unsigned long long *span)
{
    const unsigned long long span_start = SPAN ? kvq_wall_clock() : 0;      // timing-aid instantiation (kvq_profile_*)
    __shared__ __attribute__((aligned(16))) uint8_t lds[PvCfg<BITS, RG>::LDS];
    pv_dense_body<BITS, RG>(lds, (int)blockIdx.x, (int)gridDim.x, (int)blockIdx.y, KVQ_PV_DENSE_ARGS);
    if (SPAN) kvq_span_end(span, span_start);
}

// Sparse part, balanced (paper App. "Kernel Implementation Details": equal non-zeros per thread):
// lanes are outlier entries, so every lane does the same amount of work whatever the sparsity
// pattern.  A wavefront owns a run of consecutive tokens and walks it PVS_TW tokens at a time on its
// own (no workgroup barrier inside the loop): it stages the sub-range's pointers and probabilities in
// its private LDS slice, finds each entry's token by a binary search over the pointers and adds
// p[q][n] * val to the workgroup's fixed-point LDS accumulators (integer atomics).  The workgroup's
// sums go to the workspace; the reduce kernel adds them up.
// R = query heads per KV head (0: any ratio, looked up at run time); SINK: the cache keeps its first
// n_sink tokens in fp16; FUSED: `probs` holds raw scores, see below (separate instantiations: the
// plain one has no register to spare)
template <int R, bool SINK, bool FUSED, class SP>
__device__ __forceinline__ void pv_sparse_body(float *dyn, const int bx, int n_kv_heads, int n_q_heads, int64_t L, const uint32_t *__restrict__ v_ptr,
                   const SP vsp, uint32_t nnz_cap,
                   const float *__restrict__ probs, int64_t ld, float *__restrict__ spartial, PvsRuns runs, int whole_bits,
                   int n_sink, const float *__restrict__ stat_slots, int n_stat)
{
    // whole_bits: 23 and as many more as the sums of a workgroup need (pv_whole_bits)
    // FUSED: `probs` holds raw scores x; the workgroup takes every head's maximum m over its n_stat
    // slots once and scores become weights exp(x - m) on their way into the wavefront's LDS slice
    unsigned long long *sacc = (unsigned long long *)dyn;     // [n_q_heads][128] sums with 63 - whole_bits fractional bits
    float *sst = (float *)(sacc + n_q_heads * 128);           // [n_q_heads] log2(e) * maximum score (2 floats per head reserved)
    const int tid = threadIdx.x, lane = tid & 63, n_waves = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);           // scalar: loop bounds below are uniform
    float *ps = sst + 2 * n_q_heads + (size_t)wave * pvs_wave_lds_floats(n_q_heads);   // [n_q_heads][PVS_ROW]
    const int r = R ? R : n_q_heads / n_kv_heads;
    for (int j = tid; j < n_q_heads * 128; j += blockDim.x) sacc[j] = 0ull;
    bool cleared = false;      // the barrier after the clearing comes once the first loads are requested
    const int run_no = bx * n_waves + wave;
    const int64_t nb = runs.unit * ((int64_t)run_no * runs.units + (run_no < runs.longer ? run_no : runs.longer));
    int64_t ne = nb + runs.unit * (runs.units + (run_no < runs.longer ? 1 : 0));
    if (ne > L) ne = L;
    const int n_cells = n_q_heads * PVS_TW;
    // the run is cut into equal sub-ranges of at most PVS_TW tokens; the pointers of the next one are
    // requested while the current one is processed
    const int run = (nb < ne) ? (int)(ne - nb) : 0, n_sub = (run + PVS_TW - 1) / PVS_TW;
    const int sub_len = n_sub ? (run + n_sub - 1) / n_sub : 0;
    int64_t nc = nb;
    int tc = sub_len;
    uint32_t pw = 0;
    if (tc > 0) pw = v_ptr[nc + (lane < tc ? lane : tc)];
    if (FUSED) {
        // every head's maximum over its slots, four heads per wavefront at a time with their loads
        // requested together (and behind the pointer load above, so that the round trips overlap)
        for (int q0 = 4 * wave; q0 < n_q_heads; q0 += 4 * n_waves) {
            float m[4] = {KVQ_STAT_FLOOR, KVQ_STAT_FLOOR, KVQ_STAT_FLOOR, KVQ_STAT_FLOOR};
            for (int i0 = 0; i0 < n_stat; i0 += 64) {
                const int i = (i0 + lane < n_stat) ? i0 + lane : n_stat - 1;     // a repeated slot does not change a maximum
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int qh = (q0 + k < n_q_heads) ? q0 + k : q0;
                    m[k] = __builtin_fmaxf(m[k], stat_slots[(int64_t)qh * KVQ_STAT_SLOTS + i]);
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float w = kvq_wave_max(m[k]) * KVQ_LOG2E;
                if (lane == 0 && q0 + k < n_q_heads) sst[q0 + k] = w;
            }
        }
    }
    while (tc > 0) {
        const int64_t nc_next = nc + tc;
        const int tc_next = (int)((ne - nc_next < sub_len) ? (ne - nc_next) : sub_len);
        // probabilities: cell j = (query head j / 16, token j % 16); loads are straight-line (cells
        // outside the sub-range re-read its first probability and store zero)
        const int t_sink = (SINK && nc < n_sink) ? (int)(n_sink - nc) : 0;    // tokens of this sub-range kept in fp16
        float pr[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int j = lane + 64 * k, qh = j / PVS_TW, t = j % PVS_TW;
            const bool ok = j < n_cells && t < tc;
            const float x = probs[ok ? (int64_t)qh * ld + nc + t : nc];
            pr[k] = (ok && (!SINK || t >= t_sink)) ? x : 0.f;    // sink tokens: weight 0 (kept in fp16)
        }
        const uint32_t e_begin = (uint32_t)__builtin_amdgcn_readfirstlane((int)pw);
        const uint32_t e_end = (uint32_t)__builtin_amdgcn_readlane((int)pw, 63);
        uint32_t chv[PVS_U], vb[PVS_U];
        if (e_begin < e_end) {
            if (e_begin + 64u * PVS_U <= nnz_cap) kvq_sparse_load_batch<false, PVS_U>(vsp, nnz_cap, e_begin, e_end, lane, chv, vb);
            else kvq_sparse_load_batch<true, PVS_U>(vsp, nnz_cap, e_begin, e_end, lane, chv, vb);
        }
        uint32_t pw_next = 0;
        if (tc_next > 0) pw_next = v_ptr[nc_next + (lane < tc_next ? lane : tc_next)];
        if (!cleared) {          // the accumulators are clear and the statistics merged
            __syncthreads();
            cleared = true;
        }
        // (the cells' LDS addresses are recomputed from an opaque copy of the lane number: hoisted
        // out of the loop they would cost eight registers that this kernel does not have)
        int lane_o = lane;
        asm volatile("" : "+v"(lane_o));
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int j = lane_o + 64 * k, qh = j / PVS_TW, t = j % PVS_TW;
            if (j < n_cells) {
                float w = pr[k];
                if (FUSED) {
                    const float e = kvq_stat_weight(w, sst[qh]);
                    w = (t < tc && (!SINK || t >= t_sink)) ? e : 0.f;
                }
                ps[qh * PVS_ROW + t] = __builtin_ldexpf(w, 31 - whole_bits);
            }
        }
        for (int j0 = 64 * 8; j0 < n_cells; j0 += 64) {      // models with more than 32 query heads
            const int j = j0 + lane, qh = j / PVS_TW, t = j % PVS_TW;
            if (j < n_cells) {
                const bool ok = t < tc && (!SINK || t >= t_sink);
                float w = ok ? probs[(int64_t)qh * ld + nc + t] : 0.f;
                if (FUSED && ok) w = kvq_stat_weight(w, sst[qh]);
                ps[qh * PVS_ROW + t] = __builtin_ldexpf(w, 31 - whole_bits);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        int tcur = 0;
        // Every token of a sub-range normally has the same number of outliers (the append keeps
        // 2 * k_side_v per token unless the arrays ran full): entry e then belongs to token
        // (e - e_begin) / per, and the walk over the pointers (kvq_sparse_token, a third of this kernel's
        // time) is not needed.  Checked against the pointers themselves, sub-range by sub-range.
        const float perf = __builtin_truncf(((float)(e_end - e_begin) + 0.5f) * __builtin_amdgcn_rcpf((float)tc));
        const uint32_t per = (uint32_t)perf;
        const bool even = e_end - e_begin < (1u << 22) && per > 0 &&
                          __builtin_amdgcn_ballot_w64(lane <= tc && pw != e_begin + (uint32_t)lane * per) == 0ull;
        const float rper = __builtin_amdgcn_rcpf(perf);
        for (uint32_t eb = e_begin; eb < e_end; eb += 64 * PVS_U) {
            if (eb != e_begin) {                         // (the first batch was requested above)
                if (eb + 64u * PVS_U <= nnz_cap) kvq_sparse_load_batch<false, PVS_U>(vsp, nnz_cap, eb, e_end, lane, chv, vb);
                else kvq_sparse_load_batch<true, PVS_U>(vsp, nnz_cap, eb, e_end, lane, chv, vb);
            }
#pragma unroll
            for (int u = 0; u < PVS_U; ++u) {
                const uint32_t first = eb + 64u * u, e = first + (uint32_t)lane;
                if (first >= e_end) break;
                // ((x + 0.5) / per: the half keeps the quotient's rounding error, 2e-6 at most, away from an integer)
                const int t = even ? (int)(((float)(e - e_begin) + 0.5f) * rper) : kvq_sparse_token(pw, tc, tcur, first, e);
                if (e < e_end) {
                    const uint32_t ch = chv[u];
                    const float v = kvq_h2f((uint16_t)vb[u]);
                    const uint32_t kvh = ch >> 7, c = ch & 127u;
                    for (int j = 0; j < r; ++j) {
                        const uint32_t qh = kvh * r + j;
                        atomicAdd(&sacc[(R == 1) ? ch : qh * 128u + c], kvq_to_fixed_nearest(ps[qh * PVS_ROW + t] * v));
                    }
                }
            }
        }
        // the next sub-range overwrites ps: order those stores after this sub-range's reads
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        nc = nc_next;
        tc = tc_next;
        pw = pw_next;
    }
    if (!cleared) __syncthreads();       // a wavefront without tokens still meets the workgroup's barrier
    __syncthreads();
    for (int j = tid; j < n_q_heads * 128; j += blockDim.x)
        spartial[(int64_t)bx * n_q_heads * 128 + j] = __builtin_ldexpf(kvq_from_fixed<0>(sacc[j]), whole_bits - 31);
}

template <int R, bool SINK, bool FUSED, class SP>
__global__ __launch_bounds__(768) __attribute__((amdgpu_waves_per_eu(6, 6)))
void kvq_pv_sparse(int n_kv_heads, int n_q_heads, int64_t L, const uint32_t *__restrict__ v_ptr, const SP vsp,
                   uint32_t nnz_cap, const float *__restrict__ probs, int64_t ld, float *__restrict__ spartial,
                   PvsRuns runs, int whole_bits, int n_sink, const float *__restrict__ stat_slots, int n_stat)
{
    extern __shared__ __attribute__((aligned(16))) float dyn[];
    pv_sparse_body<R, SINK, FUSED, SP>(dyn, (int)blockIdx.x, n_kv_heads, n_q_heads, L, v_ptr, vsp, nnz_cap, probs, ld,
                                       spartial, runs, whole_bits, n_sink, stat_slots, n_stat);
}

// Short contexts: both as workgroups of one launch, the first n_sparse of them sparse (pv_both).  Neither kernel fills the
// chip there, and each is mostly its launch and a chain of round trips.
template <int BITS, int RG, bool FUSED, bool SPAN, class SP>
__global__ __launch_bounds__((PvCfg<BITS, RG>::NT)) void kvq_pv_both(KVQ_PV_DENSE_PARAMS, int n_sparse, int n_slabs,
                                                                    const uint32_t *__restrict__ v_ptr,
                                                                    const SP vsp, uint32_t nnz_cap,
                                                                    float *__restrict__ spartial, PvsRuns runs, int whole_bits,
                                                                    unsigned long long *span)
{
    const unsigned long long span_start = SPAN ? kvq_wall_clock() : 0;      // timing-aid instantiation (kvq_profile_*)
    extern __shared__ __attribute__((aligned(16))) float dyn[];
    const int b = (int)blockIdx.x - n_sparse;
    if (b < 0)
        pv_sparse_body<0, true, FUSED, SP>(dyn, (int)blockIdx.x, n_kv_heads, n_q_heads, L, v_ptr, vsp, nnz_cap,
                                                      probs, ld, spartial, runs, whole_bits, n_sink, stat_slots, n_stat);
    else
        pv_dense_body<BITS, RG>((uint8_t *)dyn, b % n_slabs, n_slabs, b / n_slabs, KVQ_PV_DENSE_ARGS);
    if (SPAN) kvq_span_end(span, span_start);
}

// out[q][c] = sum_slabs partial + sum_slabs zpart + sum_sslabs spartial.  Four workgroups per query
// head, each 32 channels x 32 slab groups; every sum is taken in a fixed order.
__global__ __launch_bounds__(1024) void kvq_pv_reduce(int n_q_heads, int slabs, int sslabs,
                                                      const float *__restrict__ partial,
                                                      const float *__restrict__ zpart,
                                                      const float *__restrict__ spartial, float *__restrict__ out,
                                                      int n_sink, int n_kv_heads, const uint16_t *__restrict__ sink_v,
                                                      const float *__restrict__ probs, int64_t ld,
                                                      const float *__restrict__ stat_slots, int n_stat,
                                                      const float *__restrict__ lpart)
{
    // n_sink: attention-sink tokens (already clipped to the tokens present), added from their fp16 rows;
    // stat_slots != null: `probs` holds raw scores, the partial sums are weighted by exp(x - m) (see
    // kvq_pv_dense) and the result is divided by the sum of all weights (lpart, plus the sink tokens')
    __shared__ float red[32][33];
    __shared__ float zred[32], lred[32];
    __shared__ float sm2;
    const int qh = blockIdx.x >> 2, c = (blockIdx.x & 3) * 32 + (threadIdx.x & 31), j = threadIdx.x >> 5;
    if (stat_slots && n_sink > 0 && threadIdx.x < 64) {
        float m = KVQ_STAT_FLOOR;
        for (int i = threadIdx.x; i < n_stat; i += 64) m = __builtin_fmaxf(m, stat_slots[(int64_t)qh * KVQ_STAT_SLOTS + i]);
        m = kvq_wave_max(m) * KVQ_LOG2E;
        if (threadIdx.x == 0) sm2 = m;
    }
    float s = 0.f;
    for (int k0 = j; k0 < slabs; k0 += 256) {          // eight loads in flight per thread
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = k0 + 32 * u;
            v[u] = (k < slabs) ? partial[((int64_t)k * n_q_heads + qh) * 128 + c] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (int k0 = j; k0 < sslabs; k0 += 256) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = k0 + 32 * u;
            v[u] = (k < sslabs) ? spartial[((int64_t)k * n_q_heads + qh) * 128 + c] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    red[j][threadIdx.x & 31] = s;
    if ((threadIdx.x & 31) == 0) {
        float z = 0.f;
        for (int k = j; k < slabs; k += 32) z += zpart[(int64_t)k * n_q_heads + qh];
        zred[j] = z;
        float l = 0.f;
        if (stat_slots)
            for (int k = j; k < slabs; k += 32) l += lpart[(int64_t)k * n_q_heads + qh];
        lred[j] = l;
    }
    __syncthreads();
    if (j == 0) {
        float t = 0.f, z = 0.f, l = 0.f;
#pragma unroll
        for (int i = 0; i < 32; ++i) { t += red[i][threadIdx.x & 31]; z += zred[i]; l += lred[i]; }
        float sink = 0.f;
        const int kvh = qh / (n_q_heads / n_kv_heads);
        for (int n = 0; n < n_sink; ++n) {
            float w = probs[(int64_t)qh * ld + n];
            if (stat_slots) {
                w = kvq_stat_weight(w, sm2);
                l += w;
            }
            sink = __builtin_fmaf(w, kvq_h2f(sink_v[(int64_t)n * n_kv_heads * 128 + kvh * 128 + c]), sink);
        }
        const float r = t + z + sink;
        out[qh * 128 + c] = stat_slots ? r / l : r;
    }
}

}  // namespace

int64_t kvq_pv_workspace_bytes(int n_q_heads)
{
    // no plan needs more than 512 dense + 512 sparse slabs
    // dense partials, zero-point sums, sparse partials, weight sums (fused call)
    return ((int64_t)512 * n_q_heads * 128 + (int64_t)512 * n_q_heads + (int64_t)512 * n_q_heads * 128 +
            (int64_t)512 * n_q_heads) * 4;
}

extern "C" int64_t kvq_workspace_bytes(const kvq_cache *cache, int32_t max_append)
{
    if (!cache) return 0;
    int64_t a = (int64_t)(max_append > 0 ? max_append : 1) * 4;
    // slab partials of the Value kernels, then the softmax statistics of the fused decode call
    int64_t b = kvq_pv_workspace_bytes(cache->n_q_heads) + (int64_t)cache->n_q_heads * KVQ_STAT_SLOTS * 4;
    int64_t w = a > b ? a : b;
    return (w + 255) & ~(int64_t)255;
}

extern "C" kvq_status kvq_pv_matvec(const kvq_cache *cache, const float *d_probs, int64_t ld_probs, float *d_out,
                                    void *stream)
{
    return kvq_pv_run(cache, d_probs, ld_probs, d_out, nullptr, 0, (hipStream_t)stream);
}

// Launch of the sparse kernel for either layout of the outlier entries.  ri: index of the head ratio
// among {any, 1, 2, 4, 8}.
template <class SP>
static kvq_status pv_launch_sparse(const kvq_cache *cache, const SP vsp, int ri, bool sink, bool fused,
                                   const PvPlan &plan, const float *d_probs, int64_t ld_probs, float *spartial,
                                   const float *stat_slots, int n_stat, hipStream_t s)
{
    using SparseKernel = decltype(&kvq_pv_sparse<0, false, false, SP>);
#define KVQ_PVS_ROW(R) {{kvq_pv_sparse<R, false, false, SP>, kvq_pv_sparse<R, false, true, SP>},       \
                        {kvq_pv_sparse<R, true, false, SP>, kvq_pv_sparse<R, true, true, SP>}}
    static const SparseKernel kernels[5][2][2] = {KVQ_PVS_ROW(0), KVQ_PVS_ROW(1), KVQ_PVS_ROW(2), KVQ_PVS_ROW(4),
                                                  KVQ_PVS_ROW(8)};
#undef KVQ_PVS_ROW
    const SparseKernel sparse = kernels[ri][sink][fused];
    // every instantiation's dynamic-LDS limit is raised once, to the most a plan asks for
    // (initialisation of a function-local static is thread-safe)
    static const hipError_t lds_attr = [] {
        for (auto &a : kernels)
            for (auto &b : a)
                for (SparseKernel k : b) {
                    const hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, 147456);
                    if (e != hipSuccess) return e;
                }
        return hipSuccess;
    }();
    KVQ_HIP_CHECK(lds_attr);
    if (plan.slds > 147456) return KVQ_ERR_UNSUPPORTED;
    // (Running this kernel on a second stream beside the dense one was tried: its LDS footprint
    // evicts dense workgroups from the CUs and the pair gets slower.)
    if (cache->cap_nnz_v >= ((int64_t)1 << 31)) return KVQ_ERR_UNSUPPORTED;      // byte offsets are 32-bit
    const int64_t tokens = plan.tokens_per_swave * plan.swaves;
    sparse<<<plan.sslabs, 64 * plan.swaves, plan.slds, s>>>(cache->n_kv_heads, cache->n_q_heads, cache->n_tokens_v,
                                                            cache->v_ptr, vsp, (uint32_t)cache->cap_nnz_v, d_probs,
                                                            ld_probs, spartial, PvsRuns{8, (int)(plan.tokens_per_swave / 8), 0},
                                                            pv_whole_bits(tokens, tokens, fused), cache->n_sink, stat_slots, n_stat);
    return KVQ_OK;
}

// f(bits, heads per group) as compile-time constants.
template <class F>
static auto pv_with(int bits, int rg, F f)
{
    auto with_rg = [&](auto b) {
        if (rg == 8) return f(b, std::integral_constant<int, 8>{});
        if (rg == 4) return f(b, std::integral_constant<int, 4>{});
        if (rg == 2) return f(b, std::integral_constant<int, 2>{});
        return f(b, std::integral_constant<int, 1>{});
    };
    if (bits == 2) return with_rg(std::integral_constant<int, 2>{});
    if (bits == 3) return with_rg(std::integral_constant<int, 3>{});
    return with_rg(std::integral_constant<int, 4>{});
}

// Whether the Value half of a call over cache->n_tokens_v tokens is one launch and the reduction.
static bool pv_one_launch(const kvq_cache *cache, PvBoth &p)
{
    const int rg = pv_group(cache->n_tokens_v, cache->n_q_heads, cache->n_q_heads / cache->n_kv_heads);
    return pv_both(cache, rg, pv_with(cache->bits, rg, [](auto b, auto g) { return (size_t)PvCfg<b.value, g.value>::LDS; }), p);
}

bool kvq_pv_is_one_launch(const kvq_cache *cache)
{
    PvBoth p;
    return cache->n_tokens_v > 0 && pv_one_launch(cache, p);
}

kvq_status kvq_pv_run(const kvq_cache *cache, const float *d_probs, int64_t ld_probs, float *d_out,
                      const float *stat_slots, int n_stat, hipStream_t s)
{
    kvq_status st = kvq_check_cache(cache);
    if (st != KVQ_OK) return st;
    if (!cache->loaded) return KVQ_ERR_NOT_LOADED;
    if (!d_probs || !d_out || ((uintptr_t)d_probs & 3) || ((uintptr_t)d_out & 3)) return KVQ_ERR_INVALID_ARG;
    const int64_t L = cache->n_tokens_v;
    if (ld_probs < L) return KVQ_ERR_INVALID_ARG;
    const int Hq = cache->n_q_heads, D = cache->n_kv_heads * KVQ_HEAD_DIM;
    if (!cache->workspace || cache->workspace_bytes < kvq_pv_workspace_bytes(Hq)) return KVQ_ERR_CAPACITY;
    const int r = Hq / cache->n_kv_heads;
    const int rg = pv_group(L, Hq, r);
    PvPlan plan = (L > 0) ? pv_plan(L, Hq, rg) : PvPlan{0, 0, 0, 0, 0, 0};
    float *partial = (float *)cache->workspace;
    float *zpart = partial + (int64_t)512 * Hq * 128;
    float *spartial = zpart + (int64_t)512 * Hq;
    float *lpart = spartial + (int64_t)512 * Hq * 128;
    PvBoth both;
    const bool merged = L > 0 && pv_one_launch(cache, both);
    // (the timing aid takes the launch that holds the dense kernel)
    KvqProfile &prof = kvq_profile_state();
    unsigned long long *span = nullptr;
    hipEvent_t *pev = (L > 0 && prof.enabled && prof.use_events) ? prof.ev[1][prof.count[1] % KVQ_PROFILE_RING] : nullptr;
    if (merged) {
        const int whole_bits = pv_whole_bits(both.most_tokens, plan.tokens_per_swave * plan.swaves,
                                             stat_slots != nullptr);
        plan.slabs = both.slabs;
        plan.sslabs = both.n_sparse;
        const unsigned grid = (unsigned)(both.n_sparse + both.slabs * (Hq / rg));
        span = kvq_profile_span_slot(prof, 1, grid);
        if (pev) KVQ_HIP_CHECK(hipEventRecord(pev[0], s));
        const auto launch = [&](const auto vsp) {
            using SP = std::remove_cv_t<decltype(vsp)>;
            return pv_with(cache->bits, rg, [&](auto b, auto g) {
                constexpr int BITS = decltype(b)::value, RG = decltype(g)::value;
                using Kernel = decltype(&kvq_pv_both<BITS, RG, false, false, SP>);
                static const Kernel kernels[2][2] = {{kvq_pv_both<BITS, RG, false, false, SP>, kvq_pv_both<BITS, RG, false, true, SP>},
                                                     {kvq_pv_both<BITS, RG, true, false, SP>, kvq_pv_both<BITS, RG, true, true, SP>}};
                // the dynamic-LDS limits are raised once (initialisation of a function-local static is thread-safe)
                static const hipError_t lds_attr = [] {
                    for (auto &k : kernels)
                        for (Kernel kern : k) {
                            const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, PV_BOTH_LDS);
                            if (e != hipSuccess) return e;
                        }
                    return hipSuccess;
                }();
                if (lds_attr != hipSuccess) return lds_attr;
                kernels[stat_slots != nullptr][span != nullptr]<<<grid, (PvCfg<BITS, RG>::NT), both.lds, s>>>(
                    cache->params, D, cache->n_kv_heads, Hq, cache->cap_tokens, L, cache->v_codes, cache->v_sz, d_probs, ld_probs,
                    partial, zpart, plan.tiles, cache->n_sink, stat_slots, n_stat, lpart, both.n_sparse, both.slabs, cache->v_ptr,
                    vsp, (uint32_t)cache->cap_nnz_v, spartial, both.runs, whole_bits, span);
                return hipSuccess;
            });
        };
        KVQ_HIP_CHECK(cache->nnz_block_shift ? launch(kvq_blocked_v(cache)) : launch(kvq_flat_v(cache)));
    }
    if (L > 0 && !merged) {
        const bool sink = cache->n_sink > 0;
        const int ri = (r == 1) ? 1 : (r == 2) ? 2 : (r == 4) ? 3 : (r == 8) ? 4 : 0;
        const bool fused = stat_slots != nullptr;
        st = cache->nnz_block_shift
                 ? pv_launch_sparse(cache, kvq_blocked_v(cache), ri, sink, fused, plan, d_probs, ld_probs, spartial,
                                    stat_slots, n_stat, s)
                 : pv_launch_sparse(cache, kvq_flat_v(cache), ri, sink, fused, plan, d_probs, ld_probs, spartial,
                                    stat_slots, n_stat, s);
        if (st != KVQ_OK) return st;

        dim3 grid((unsigned)plan.slabs, (unsigned)(Hq / rg));
#define LAUNCH_PV(B, G)                                                                                        \
    do {                                                                                                       \
        auto kern = span ? kvq_pv_dense<B, G, true> : kvq_pv_dense<B, G, false>;                               \
        kern<<<grid, (PvCfg<B, G>::NT), 0, s>>>(cache->params, D, cache->n_kv_heads, Hq, cache->cap_tokens, L,   \
                                              cache->v_codes, cache->v_sz, d_probs, ld_probs, partial, zpart,  \
                                              plan.tiles, cache->n_sink, stat_slots, n_stat, lpart, span);     \
    } while (0)
#define LAUNCH_PV_B(B)                                                                                         \
    do {                                                                                                       \
        if (rg == 8) LAUNCH_PV(B, 8);                                                                          \
        else if (rg == 4) LAUNCH_PV(B, 4);                                                                     \
        else if (rg == 2) LAUNCH_PV(B, 2);                                                                     \
        else LAUNCH_PV(B, 1);                                                                                  \
    } while (0)
        span = kvq_profile_span_slot(prof, 1, (int64_t)grid.x * grid.y);
        if (pev) KVQ_HIP_CHECK(hipEventRecord(pev[0], s));
        if (cache->bits == 2) LAUNCH_PV_B(2);
        else if (cache->bits == 3) LAUNCH_PV_B(3);
        else LAUNCH_PV_B(4);
#undef LAUNCH_PV_B
#undef LAUNCH_PV
    }
    if (pev) KVQ_HIP_CHECK(hipEventRecord(pev[1], s));
    if (L > 0 && prof.enabled) ++prof.count[1];
    const int ns = (int)(cache->n_sink < L ? cache->n_sink : L);
    kvq_pv_reduce<<<4 * Hq, 1024, 0, s>>>(Hq, plan.slabs, plan.sslabs, partial, zpart, spartial, d_out, ns,
                                          cache->n_kv_heads, cache->sink_v, d_probs, ld_probs, stat_slots, n_stat, lpart);
    KVQ_HIP_CHECK(hipGetLastError());
    return KVQ_OK;
}
