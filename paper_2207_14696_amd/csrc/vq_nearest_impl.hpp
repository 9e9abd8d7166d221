// Nearest codebook entry on the matrix cores (Sec. 3.2's search; the encoder and the assignment
// step of the codebook training use it).
//
// The result is defined bit by bit: the entry with the smallest fp32 distance, columns in order,
// every operation rounded by itself, ties to the lowest index (cosine: the largest fp32 dot
// product times the entry's reciprocal norm).  Evaluating that rule for every entry costs 3
// vector instructions per column and entry and leaves the matrix cores idle.  Here they do the
// search: s = |c|^2/2 - x.c (cosine: -x.c/|c|) for 32 rows x 32 entries at a time, both factors
// split into two half-precision pieces (hi + lo, 22 bits).  Per 8 columns x.c_hi is one MFMA of
// K = 16 (the row's high pieces in the lower lanes, its low ones in the upper) and x_hi.c_lo half of
// one; the other half of an odd last one carries |c|^2/2 in three pieces (with an even number of
// groups of 8 columns, or without the entries in LDS, the accumulators start from it).  A lane
// keeps, per row, the best and the second best *cell* (8 entries: half of the accumulators of a
// tile), which costs 6 vector instructions per 8 scores; the 8 entries of the winning cell are then
// scored in fp32.  Each of the two decisions is certain to be the rule's own when the second best is
// further away than the errors of both evaluations together (derived at vq_margin and
// vq_cell_margin below); a row for which it is not - near ties, values outside the range the split
// holds - is searched by the rule over the whole codebook, by the wave together, or lane by lane
// when many rows of a wave need it; where most rows do, the scores are left out (search_costs below:
// at no share of such rows is that dearer than the plain search by more than a fifth, but parts of 4
// columns, which count as 8 here: 96 x 256 x 4 464 us by the plain search, 130 with no such row, 570 at a fifth, 770 at worst).
// The codes are therefore the same as the plain search gives, for any input.
//
// What bounds it: vector instructions and power.  Of 479 per 64 rows and part 200 are the running
// minima over 256 entries, 100 the scores inside the cell, 45 the split of x, 32 the products, at
// 78 % of the issue rate; the clock falls to 1.8 GHz under it, so that every instruction and LDS
// read taken out counts, and a better overlap alone does not.  262 144 rows of 96 parts x 256 entries
// x 8 columns: 535 us; with all four products of the pieces, |c|^2/2 read from LDS for every tile
// and cells across two tiles (570 instructions, 77 LDS reads instead of 39) 650; the plain search
// 3111 us.  Cells of 4 entries cost as much more in minima as they save in scores, of 16 more.
//
// Training adds each part to its entry's sum in LDS.  The sums are kept in 64 bits: an LDS
// float add takes 196 cycles per wave here whatever the addresses, a double add 22 (integer: 8).
// A workgroup writes the sums of its sets of rows (RowSets) to the workspace and a second kernel adds
// them up in the sets' order (global float adds onto the same few addresses ran at 22.6 G/s, a quarter of
// the round).  One round over 65 536 rows of that shape: 167 us (with the search as it was, see above,
// 200; with the rows dealt evenly instead of in sets, and codebooks that depend on how many
// workgroups there are, 164; plain search and fp32 adds 1030).
#pragma once

#include "vq_nearest.hpp"

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace bf {

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float16v __attribute__((ext_vector_type(16)));

template <typename T>
struct VqNearestArgs {
    const T *x;             // [rows x D]
    int64_t rows;
    int D, w, len, P, cbytes;
    int bvec;               // 4 columns of a part, of an entry are loaded at once
    int lane_rows, plain_rows;  // see search_costs
    int NT;                 // tiles of 32 entries
    int ny;                 // workgroups per part
    int more;               // (the encoder) of the last part on top of these
    int64_t chunk;          // rows of each, a whole number of waves
    int64_t last_chunk;     // (the encoder) the last part's
    int strip_log2, sets, sub;  // (training) see RowSets
    const float *rnorm;     // [P][len], cosine metric
    float margin, cell_margin;  // see vq_margin
    uint32_t cell_mask;     // low bits of a score that hold a cell's number
    int64_t rb, pb;         // (the encoder) from one row's index, one part's to the next
    int one_set;            // (training) every workgroup adds to one set of sums, all zeros
    void *sums;             // [sets][sub][P][w][len], in 64 bits where sub > 1, else 32
    uint32_t *counts;       // [sets][sub][P][len]
    double *distortion;     // [workgroups], with one_set: the round's
};

// codebooks of fewer values (entries x columns; parts of 4 columns or more; with few rows x parts) and
// wider parts stay with the plain search, see vq_nearest_takes
constexpr int kNearestMinBook = 512, kNearestMinBookAny = 64, kNearestMinBookFew = 384;
constexpr int kNearestMaxWidth = 32;
constexpr int kCuLds = 160 * 1024;
// strips that a wave searches by the rule once its rows tie, before it tries the scores again
constexpr int kPlainStrips = 7;

constexpr float kPadScore = 1e30f;   // score of the entries that fill up the last tile
// Layout in LDS.  Entry pieces of a tile, in units of 8 halves: [high pieces: G x 32 | low pieces:
// G x 32 | with NORM |c|^2/2 in three pieces and a fourth that only padding entries have, 4 halves
// an entry].  Entries: 4 of them, then 4 floats (|c|^2/2; cosine: 1/|c|); after 4 such groups 4
// floats of padding, so that lanes that read different ones meet in few banks.
__host__ __device__ constexpr bool norm_slot(int G, bool ent) { return ent && G % 2 == 1; }
__host__ __device__ constexpr int tile_units(int G, bool ent) { return 64 * G + (norm_slot(G, ent) ? 16 : 0); }
__host__ __device__ constexpr int group_floats(int G) { return 4 * 8 * G + 4; }
__host__ __device__ constexpr int groups4_floats(int G) { return 4 * group_floats(G) + 4; }
// what the pieces of |c|^2/2 (at most 2^26) are multiplied with; the fourth makes 2^31
constexpr float kNormUnit1 = 4096.0f, kNormUnit2 = 2.0f, kPadUnit = 32768.0f, kPadPiece = 65504.0f;
constexpr float kMinHalf = 0x1p-14f;  // smallest normal half
constexpr int kScaleExp = 11;        // largest magnitude of a part's codebook: [2^10, 2^11)
constexpr float kMaxNorm2 = 1073741824.0f;  // rows with a scaled |x|^2 of 2^30 or more go by the rule

// One instruction for up to three operands, and none to quiet NaNs first (fminf needs one each); a
// NaN wins, which the caller's comparison with the margin then sees.
__device__ inline float minimum(float a, float b) { return __builtin_elementwise_minimum(a, b); }

// a minus the half in the low / high bits of h: exact where that is a's high piece, and one instruction
// (the compiler makes a conversion and a subtraction of it)
__device__ inline float less_low(float a, uint32_t h) {
    float d;
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(d) : "v"(h), "v"(a));
    return d;
}
__device__ inline float less_high(float a, uint32_t h) {
    float d;
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(h), "v"(a));
    return d;
}

// The rule, column by column.
template <int METRIC>
__device__ inline float rule_step(float acc, float x, float c) {
    if constexpr (METRIC == BIFEAT_VQ_COSINE) return __fadd_rn(acc, __fmul_rn(x, c));
    const float diff = __fsub_rn(x, c);
    return __fadd_rn(acc, __fmul_rn(diff, diff));
}

// One row's distance to one entry by the rule (smaller = better; cosine: the negated score).
template <int WP, int METRIC>
__device__ inline float rule_value(const float (&x)[WP], const float (&c)[WP], float rn) {
    float acc = 0.0f;
#pragma unroll
    for (int d = 0; d < WP; d++) acc = rule_step<METRIC>(acc, x[d], c[d]);
    if constexpr (METRIC == BIFEAT_VQ_COSINE) return -__fmul_rn(acc, rn);
    else return acc;
}

// waves of a SIMD, workgroups of a CU with a copy of the entries in LDS (9 to 16 columns: with 2 waves
// the whole search by the rule, 48 x 256 x 16, took 846 us instead of 770, the scores 181 instead of 166)
// (one workgroup of 512 threads: 2)
constexpr int nearest_waves(int G, bool ent, int TH = 256) { return G == 1 ? 4 : G == 2 && ent && TH == 256 ? 3 : 2; }

template <typename T, int G, int METRIC, bool ENT, bool TRAIN, int TH>
__global__ __launch_bounds__(TH, nearest_waves(G, ENT, TH)) void vq_nearest_kernel(
    VqNearestArgs<T> a, const float *__restrict__ cb, uint8_t *__restrict__ codes) {
    constexpr int WP = 8 * G;          // columns of a part, padded with zeros
    constexpr int WAVES = TH / 64;
    constexpr int GROUP = group_floats(G), GROUPS4 = groups4_floats(G), UNITS = tile_units(G, ENT);
    constexpr bool COS = METRIC == BIFEAT_VQ_COSINE;
    // whether |c|^2/2 comes with the product or is what the accumulators start from
    constexpr bool NORM = norm_slot(G, ENT);
    constexpr int LO = (G + 1) / 2;    // products with low pieces, two groups of columns at a time
    extern __shared__ uint4 s_raw[];
    // [entry pieces: NT x UNITS x 16 bytes, NORM: 16 more of zeros, else the scores' constant: NT x 32
    // floats | entries | sums by column, counts]
    half8 *s_frag = reinterpret_cast<half8 *>(s_raw);
    float *s_half = reinterpret_cast<float *>(s_frag + (size_t)a.NT * UNITS);
    float *s_ent = s_half + (NORM ? 4 : a.NT * 32);
    // (every piece above is a multiple of 4 floats)
    double *s_sum = reinterpret_cast<double *>(s_ent + (ENT ? a.NT * 2 * GROUPS4 : 0));
    uint32_t *s_cnt = reinterpret_cast<uint32_t *>(s_sum + (TRAIN ? a.len * a.w : 0));
    __shared__ unsigned s_cmax, s_c2max;
    __shared__ int s_bad;
    __shared__ double s_dist;

    // workgroups are dealt to the XCDs in turn: consecutive logical ids (the parts of one strip
    // of rows, which share memory lines of x and of the codes) belong on one XCD
    const unsigned per_xcd = gridDim.x >> 3;
    const unsigned id = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    const unsigned even = (unsigned)(a.P * a.ny);
    if (id >= even + (TRAIN ? 0u : (unsigned)a.more)) return;
    const bool extra = !TRAIN && id >= even;
    const int part = extra ? a.P - 1 : (int)(id % (unsigned)a.P), by = extra ? (int)(id - even) + a.ny : (int)(id / (unsigned)a.P);
    const int64_t chunk = !TRAIN && part == a.P - 1 ? a.last_chunk : a.chunk;
    const int lane = threadIdx.x & 63;
    const int half = lane >> 5;
    const int w = a.w, len = a.len;
    const float *part_cb = cb + (int64_t)part * len * w;
    const float *part_rn = COS ? a.rnorm + (int64_t)part * len : nullptr;

    // ---- the part's scale: a power of two that brings its largest magnitude to [2^10, 2^11)
    if (threadIdx.x == 0) { s_cmax = 0u; s_c2max = 0u; s_bad = 0; s_dist = 0.0; }
    __syncthreads();
    float scale;
    {
        float m = 0.0f;
        bool bad = false;
        auto take = [&](float c) {
            bad |= !(fabsf(c) <= 0x1p40f);
            m = fmaxf(m, fabsf(c));
        };
        if (a.bvec) {
            for (int i = threadIdx.x; i < len * w / 4; i += TH) {
                const float4 c = reinterpret_cast<const float4 *>(part_cb)[i];
                take(c.x); take(c.y); take(c.z); take(c.w);
            }
        } else {
            for (int i = threadIdx.x; i < len * w; i += TH) take(part_cb[i]);
        }
        if constexpr (COS)
            for (int i = threadIdx.x; i < len; i += TH) bad |= !(part_rn[i] <= 0x1p40f);
        atomicMax(&s_cmax, __float_as_uint(m));
        if (bad) s_bad = 1;
        __syncthreads();
        const float cmax = __uint_as_float(s_cmax);
        int e = 0;
        frexpf(cmax, &e);
        scale = COS ? 1.0f : ldexpf(1.0f, kScaleExp - e);
        // outside this range distances by the rule could overflow or lose bits to underflow
        if (threadIdx.x == 0 && !(cmax >= 0x1p-40f)) s_bad = 1;
    }
    if constexpr (TRAIN) {
        for (int i = threadIdx.x; i < len * w; i += TH) s_sum[i] = 0.0;
        for (int i = threadIdx.x; i < len; i += TH) s_cnt[i] = 0u;
    }

    // entry e in LDS, and its |c|^2/2 (cosine: 1/|c|); from a multiple of 4 on 4 follow each other
    auto ent_at = [&](int e) { return s_ent + (e >> 4) * GROUPS4 + ((e >> 2) & 3) * GROUP + (e & 3) * WP; };
    auto norm_at = [&](int e) { return s_ent + (e >> 4) * GROUPS4 + ((e >> 2) & 3) * GROUP + 4 * WP + (e & 3); };
    // entry e from memory (columns past w: zeros)
    auto read_entry = [&](int e, float (&c)[WP]) {
        const float *src = part_cb + (int64_t)e * w;
        if (a.bvec) {
#pragma unroll
            for (int k = 0; k < WP / 4; k++) {
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                if (4 * k < w) v = reinterpret_cast<const float4 *>(src)[k];
                c[4 * k] = v.x; c[4 * k + 1] = v.y; c[4 * k + 2] = v.z; c[4 * k + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int d = 0; d < WP; d++) c[d] = d < w ? src[d] : 0.0f;
        }
    };
    const float unscale = 1.0f / (scale * scale);
    // the entries into LDS, a thread prepares one at a time
    {
        if (NORM && threadIdx.x < 4) s_half[threadIdx.x] = 0.0f;
        for (int e = threadIdx.x; e < a.NT * 32; e += TH) {
            const bool real = e < len;
            const float rn = COS ? (real ? part_rn[e] : 0.0f) : 0.0f;
            float s2 = 0.0f;
            half8 *tile = s_frag + (e >> 5) * UNITS;
            float cv[WP];
#pragma unroll
            for (int d = 0; d < WP; d++) cv[d] = 0.0f;
            if (real) read_entry(e, cv);
#pragma unroll
            for (int g = 0; g < G; g++) {
                half8 hi, lo;
#pragma unroll
                for (int j = 0; j < 8; j++) {
                    const int d = 8 * g + j;
                    const float c = cv[d];
                    float cs = COS ? c * (rn * 1024.0f) : c * scale;
                    // one fp32 value for both pieces: the compiler may otherwise fold the product
                    // into one of the conversions and round the pieces from different values
                    asm volatile("" : "+v"(cs));
                    s2 += cs * cs;
                    hi[j] = (_Float16)(-cs);
                    lo[j] = (_Float16)(-cs - (float)hi[j]);
                }
                tile[32 * g + (e & 31)] = hi;
                tile[32 * (G + g) + (e & 31)] = lo;
            }
            if constexpr (ENT) {
#pragma unroll
                for (int d = 0; d < WP; d += 4)
                    *reinterpret_cast<float4 *>(ent_at(e) + d) = make_float4(cv[d], cv[d + 1], cv[d + 2], cv[d + 3]);
            }
            const float half2 = COS ? 0.0f : 0.5f * s2;
            if constexpr (NORM) {
                // a piece that would not be a normal half is left to the next one
                const float n1 = half2 * (1.0f / kNormUnit1);
                const _Float16 p1 = n1 < kMinHalf ? (_Float16)0.0f : (_Float16)n1;
                const float r1 = half2 - (float)p1 * kNormUnit1, n2 = r1 * (1.0f / kNormUnit2);
                const _Float16 p2 = fabsf(n2) < kMinHalf ? (_Float16)0.0f : (_Float16)n2;
                const _Float16 p3 = (_Float16)(r1 - (float)p2 * kNormUnit2);
                _Float16 *norm = reinterpret_cast<_Float16 *>(tile + 64 * G) + 4 * (e & 31);
                norm[0] = real ? p1 : (_Float16)0.0f;
                norm[1] = real ? p2 : (_Float16)0.0f;
                norm[2] = real ? p3 : (_Float16)0.0f;
                norm[3] = real ? (_Float16)0.0f : (_Float16)kPadPiece;
            } else {
                s_half[e] = real ? half2 : kPadScore;
            }
            if constexpr (ENT)
                *norm_at(e) = COS ? rn : real ? half2 * unscale : kPadScore;
            if (!COS) atomicMax(&s_c2max, __float_as_uint(s2));
        }
    }
    __syncthreads();
    const bool part_bad = s_bad != 0;
    const float c2max = __uint_as_float(s_c2max) * 1.0001f;
    uint32_t keep = ~a.cell_mask;
    asm volatile("" : "+v"(keep));  // in a vector register: mask and cell number are then one instruction

    // entry e as the rule sees it (columns past w: zeros)
    auto entry = [&](int e, float (&c)[WP], float &rn) {
        if constexpr (ENT) {
            const float4 *src = reinterpret_cast<const float4 *>(ent_at(e));
#pragma unroll
            for (int k = 0; k < WP / 4; k++) {
                const float4 v = src[k];
                c[4 * k] = v.x; c[4 * k + 1] = v.y; c[4 * k + 2] = v.z; c[4 * k + 3] = v.w;
            }
            rn = COS ? *norm_at(e) : 0.0f;
        } else {
            read_entry(e, c);
            rn = COS ? part_rn[e] : 0.0f;
        }
    };

    [[maybe_unused]] const half8 norm_units = {(_Float16)kNormUnit1, (_Float16)kNormUnit2, (_Float16)1.0f,
                                               (_Float16)kPadUnit, 0, 0, 0, 0};
    // (in units of 8 bytes, from the last group's low pieces)
    [[maybe_unused]] const int last_piece = half ? 32 + lane : 2 * lane;
    float dsum = 0.0f;
    // Rows whose entries tie (0/1 features) are open more often than not; from a share on where the
    // scores and the rows searched one by one cost more than all rows by the rule, each lane for its
    // own, they are searched that way.  The entries for that come from LDS.  With a copy of them there
    // a wave decides for itself, and tries the scores again every so many strips.  Without one they
    // take the place of the pieces (32 x 8G floats are as large as a tile's pieces), so the workgroup
    // decides, now and then, and for good; every wave of it walks the same strips.
    bool plain = false;
    int plain_left = 0;
    const float *s_plain = reinterpret_cast<const float *>(s_frag);
    auto plain_book = [&](int e) {  // entries e .. e + 3, e a multiple of 4
        return ENT ? ent_at(e) : s_plain + e * WP;
    };
    constexpr int ROWS = WAVES * 64;
    const int have = min(w, a.D - part * w);  // columns that the table has
    auto load_row = [&](const T *src, float (&v)[WP]) {
        // (rows that begin anywhere too: with a load a column, each of 64 lines, 141 483 half-precision rows of 11 x 64 x
        // 16 by cosine, 174 columns, took 120 us, 49 so; 83 639 of 10 x 256 x 32, 301 columns, 157 and 75)
        if (a.bvec) {
            // (compared anew for every row: kept, the outcomes take more scalar registers than there are; half precision is
            // converted behind the branches, which would otherwise wait for their loads)
            int left = have;
            asm volatile("" : "+s"(left));
            decltype(four_any(src)) q[WP / 4];
            // (whole parts without a branch a load: training 65 536 rows of 8 x 256 x 16 505 -> 495 us, 48 x 256 x 16 1655 -> 1646, encoding
            // 100 000 of 76 x 64 x 8 100 -> 88; but training 1000 rows of 4 x 64 x 8 143 -> 146.5)
            if ((!TRAIN || WP > 8) && left >= WP) {
#pragma unroll
                for (int k = 0; k < WP / 4; k++) q[k] = four_any(src + 4 * k);
            } else {
#pragma unroll
                for (int k = 0; k < WP / 4; k++) q[k] = four_first(src + 4 * k, left - 4 * k);
            }
#pragma unroll
            for (int k = 0; k < WP / 4; k++) {
                const float4 f = to_float4(q[k]);
                v[4 * k] = f.x; v[4 * k + 1] = f.y; v[4 * k + 2] = f.z; v[4 * k + 3] = f.w;
            }
        } else {
#pragma unroll
            for (int d = 0; d < WP; d++) v[d] = d < have ? load1(src + d) : 0.0f;
        }
    };
    // (a row past the last one reads the last one; 64-bit products only where a strip is not whole.  In
    // training rows are counted within a set)
    const T *const first_row = a.x + (int64_t)part * w;
    int set = TRAIN ? by / a.sub : 0;
    const int sub = TRAIN ? by - set * a.sub : by;
    auto clamped = [&](int64_t r0) {
        int64_t row = r0 + threadIdx.x;
        if constexpr (TRAIN) row = set_row(set, a.sets, a.strip_log2, row);
        return first_row + (row < a.rows ? row : a.rows - 1) * a.D;
    };
    const T *next;
    auto load_next = [&](int64_t r0, float (&v)[WP]) {
        next = !TRAIN && r0 + 2 * ROWS <= a.rows ? next + (int64_t)ROWS * a.D : clamped(r0 + ROWS);
        load_row(next, v);
    };
    [[maybe_unused]] int strip = 0;
    [[maybe_unused]] uint8_t *out = codes;
    do {
        const int64_t begin = sub * chunk;
        const int64_t end = min(TRAIN ? set_rows(set, a.sets, a.strip_log2, a.rows) : a.rows, begin + chunk);
        if constexpr (!TRAIN) out += (begin + threadIdx.x) * a.rb + part * a.pb;
        next = clamped(begin);
        float xn[WP];
        load_row(next, xn);
        for (int64_t r0 = begin; r0 < end; r0 += ROWS) {
            // ---- 64 rows per wave, one per lane: the sub-vector split into pieces, which the halves of
            // the wave then hold for both sets of 32 rows
            const bool valid = (int64_t)threadIdx.x < end - r0;
            // (a wave without rows has nothing to do, but the workgroup decides together without a copy of
            // the entries)
            if (ENT && __builtin_amdgcn_readfirstlane(threadIdx.x) >= end - r0) break;
            float xr[WP];
#pragma unroll
            for (int d = 0; d < WP; d++) xr[d] = xn[d];
            int code = 0;
            int all_code = 0;
            float all_value = INFINITY;
            auto search_all = [&]() {
                // EP entries at a time, each read by all lanes from one address, the next ones while
                // these are evaluated (those past the last one are in bounds and not used)
                constexpr int EP = WP <= 16 ? 4 : 2;
                float4 q[2][EP][WP / 4];
                auto read = [&](float4 (&to)[EP][WP / 4], int e0) {
                    const float *src = plain_book(e0 & ~3) + (EP < 4 ? (e0 & 3) * WP : 0);
#pragma unroll
                    for (int k = 0; k < EP; k++)
#pragma unroll
                        for (int i = 0; i < WP / 4; i++) to[k][i] = reinterpret_cast<const float4 *>(src + k * WP)[i];
                };
                // (the entries' sums side by side: with two waves a SIMD nothing else hides an addition)
                auto take = [&](const float4 (&of)[EP][WP / 4], int e0, int n) {
                    float v[EP];
                    [[maybe_unused]] float rn[EP];
#pragma unroll
                    for (int k = 0; k < EP; k++) v[k] = 0.0f;
                    if constexpr (COS) {
                        const float *src = ENT ? norm_at(e0) : part_rn + e0;
#pragma unroll
                        for (int k = 0; k < EP; k++) rn[k] = src[ENT || k < n ? k : 0];
                    }
#pragma unroll
                    for (int i = 0; i < WP / 4; i++)
#pragma unroll
                        for (int k = 0; k < EP; k++) {
                            v[k] = rule_step<METRIC>(v[k], xr[4 * i], of[k][i].x);
                            v[k] = rule_step<METRIC>(v[k], xr[4 * i + 1], of[k][i].y);
                            v[k] = rule_step<METRIC>(v[k], xr[4 * i + 2], of[k][i].z);
                            v[k] = rule_step<METRIC>(v[k], xr[4 * i + 3], of[k][i].w);
                        }
#pragma unroll
                    for (int k = 0; k < EP; k++) {
                        if (k >= n) break;
                        if constexpr (COS) v[k] = -__fmul_rn(v[k], rn[k]);
                        if (v[k] < all_value) { all_value = v[k]; all_code = e0 + k; }
                    }
                };
                const int last = a.NT * 32 - EP;
                int e0 = 0;
                read(q[0], 0);
                for (; e0 + 2 * EP <= len; e0 += 2 * EP) {
                    read(q[1], e0 + EP);
                    take(q[0], e0, EP);
                    read(q[0], min(e0 + 2 * EP, last));
                    take(q[1], e0 + EP, EP);
                }
                if (e0 < len) take(q[0], e0, len - e0);
                if (e0 + EP < len) {
                    read(q[1], e0 + EP);
                    take(q[1], e0 + EP, len - e0 - EP);
                }
            };
            if (plain || plain_left > 0) {
                plain_left--;
                load_next(r0, xn);
                search_all();
                code = all_code;
            } else {
            float f = scale;
            bool bad = part_bad, zero = false;
            if constexpr (COS) {  // the best entry does not depend on the row's length
                float m = 0.0f;
#pragma unroll
                for (int d = 0; d < WP; d++) m = fmaxf(m, fabsf(xr[d]));
                int e = 0;
                frexpf(m, &e);
                zero = m == 0.0f;
                bad |= !zero && !(m >= 0x1p-50f && m <= 0x1p50f);
                f = zero || bad ? 1.0f : ldexpf(1.0f, kScaleExp - e);
            }
            float s2 = 0.0f;
            // products with the high pieces of the entries: the lower lanes multiply them with the row's high
            // pieces, the upper ones with its low pieces; with their low pieces: two groups of columns side by
            // side, of an odd last group beside |c|^2/2 (or the low pieces once more)
            half8 xh[2][G], xl[2][LO];
            {
                uint32_t hi[4 * G], lo[4 * G];
#pragma unroll
                for (int j = 0; j < 4 * G; j++) {
                    const float u = xr[2 * j] * f, v = xr[2 * j + 1] * f;
                    const auto h = __builtin_amdgcn_cvt_pkrtz(u, v);
                    hi[j] = __builtin_bit_cast(uint32_t, h);
                    // |x|^2 from the high pieces, short of it by less than 2^-9 of itself (vq_margin)
                    s2 = __builtin_amdgcn_fdot2(__builtin_bit_cast(half2v, h), __builtin_bit_cast(half2v, h), s2, false);
                    lo[j] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(less_low(u, hi[j]), less_high(v, hi[j])));
                }
                // one exchange of halves of two registers: [rows 0..31 of both], [rows 32..63 of both]
                auto both = [&](half8 (&x0), half8 (&x1), const uint32_t *p, const uint32_t *q) {
                    uint32_t set[2][4];
#pragma unroll
                    for (int j = 0; j < 4; j++) {
                        const auto e = __builtin_amdgcn_permlane32_swap(p[j], q[j], false, false);
                        set[0][j] = e[0];
                        set[1][j] = e[1];
                    }
                    __builtin_memcpy(&x0, set[0], 16);
                    __builtin_memcpy(&x1, set[1], 16);
                };
#pragma unroll
                for (int g = 0; g + 1 < G; g += 2) both(xl[0][g / 2], xl[1][g / 2], hi + 4 * g, hi + 4 * g + 4);
#pragma unroll
                for (int g = 0; g < G; g++) both(xh[0][g], xh[1][g], hi + 4 * g, lo + 4 * g);
                if constexpr (G % 2 == 1) {
#pragma unroll
                    for (int s = 0; s < 2; s++) {
                        xl[s][LO - 1] = xh[s][G - 1];
                        if constexpr (NORM)
                            if (half) xl[s][LO - 1] = norm_units;
                    }
                }
            }
            bad |= !(s2 < kMaxNorm2);  // also NaN
            const float big = COS ? sqrtf(s2) * 1024.5f : s2 + c2max;
            const float margin = bad ? INFINITY : big * a.margin;
            // (the cosine cell's scores are in units of |x|, unscaled)
            const float cell_margin = COS ? sqrtf(s2) * a.cell_margin / f : big * unscale * a.cell_margin;
            if constexpr (COS) zero = zero && s2 == 0.0f && !part_bad;  // not a NaN that fmaxf passed over
            // the next strip's rows travel during this strip's search
            load_next(r0, xn);
            float best[2] = {3e38f, 3e38f}, second[2] = {3e38f, 3e38f};
            {
                const int nt = a.NT;
                // A set's minima are taken while the matrix cores work on the other set: the next tile's
                // product is started as soon as its accumulators are free, its operands having been
                // read from LDS one half-step earlier.
                half8 eh[G], el[LO];
                float16v c;
                auto fetch = [&](int t) {
                    const half8 *tile = s_frag + t * UNITS;
                    if constexpr (!NORM) {
#pragma unroll
                        for (int q = 0; q < 4; q++) {
                            const float4 n = *reinterpret_cast<const float4 *>(s_half + t * 32 + 8 * q + 4 * half);
                            c[4 * q] = n.x; c[4 * q + 1] = n.y; c[4 * q + 2] = n.z; c[4 * q + 3] = n.w;
                        }
                    }
#pragma unroll
                    for (int g = 0; g < G; g++) eh[g] = tile[32 * g + (lane & 31)];
#pragma unroll
                    for (int g = 0; g < G / 2; g++) el[g] = tile[32 * G + 64 * g + lane];
                    if constexpr (NORM) {
                        // (the upper lanes: their entry's 8 bytes and the 8 after them, which meet zeros)
                        const uint2 *p = reinterpret_cast<const uint2 *>(tile + 32 * (2 * G - 1)) + last_piece;
                        const uint2 v0 = p[0], v1 = p[1];
                        const uint4 v = make_uint4(v0.x, v0.y, v1.x, v1.y);
                        __builtin_memcpy(&el[LO - 1], &v, 16);
                    } else if constexpr (G % 2 == 1) {
                        el[LO - 1] = tile[32 * (2 * G - 1) + (lane & 31)];
                    }
                };
                float16v acc[2];
                auto product = [&](int s) {
                    if constexpr (NORM) {
#pragma unroll
                        for (int i = 0; i < 16; i++) acc[s][i] = 0.0f;
                    } else {
                        acc[s] = c;
                    }
#pragma unroll
                    for (int g = 0; g < G; g++)
                        acc[s] = __builtin_amdgcn_mfma_f32_32x32x16_f16(eh[g], xh[s][g], acc[s], 0, 0, 0);
#pragma unroll
                    for (int g = 0; g < LO; g++)
                        acc[s] = __builtin_amdgcn_mfma_f32_32x32x16_f16(el[g], xl[s][g], acc[s], 0, 0, 0);
                };
                // (the runner-up of a tile's two keys waits for the next tile's: one instruction for both; with
                // more columns the registers are missed elsewhere)
                constexpr bool PAIRED = G == 1;
                float runner[2] = {3e38f, 3e38f};
                auto minima = [&](int s, int t, auto odd) {
                    float key[2];
#pragma unroll
                    for (int q = 0; q < 2; q++) {
                        uint32_t number = (uint32_t)(2 * t + q);
                        asm volatile("" : "+s"(number));  // one scalar: the compiler would add it up per lane
                        float m = acc[s][8 * q];
#pragma unroll
                        for (int i = 1; i < 7; i += 2) m = minimum(minimum(m, acc[s][8 * q + i]), acc[s][8 * q + i + 1]);
                        m = minimum(m, acc[s][8 * q + 7]);
                        // the cell's number replaces the low bits of its score
                        key[q] = __uint_as_float((__float_as_uint(m) & keep) | number);
                    }
                    const float r = __builtin_amdgcn_fmed3f(best[s], key[0], key[1]);
                    if constexpr (!PAIRED) second[s] = minimum(second[s], r);
                    else if constexpr (odd.value) second[s] = minimum(minimum(second[s], runner[s]), r);
                    else runner[s] = r;
                    best[s] = minimum(minimum(best[s], key[0]), key[1]);
                };
                fetch(0);
                product(0);
                product(1);
                if constexpr (!NORM) asm volatile("" : : "v"(c));
                fetch(min(1, nt - 1));
                auto tile = [&](int t, auto odd) {
                    // (c outlives both products of a step: one of them would otherwise take over its
                    // registers, and 32 copies would put things back in place)
                    __builtin_amdgcn_sched_barrier(0);
                    minima(0, t, odd);
                    __builtin_amdgcn_sched_barrier(0);
                    product(0);
                    minima(1, t, odd);
                    __builtin_amdgcn_sched_barrier(0);
                    product(1);
                    if constexpr (!NORM) asm volatile("" : : "v"(c));
                    fetch(min(t + 2, nt - 1));
                };
                int t = 0;
                if constexpr (!PAIRED)
                    for (; t + 1 < nt; t++) tile(t, std::false_type());
                for (; PAIRED && t + 2 < nt; t += 2) {
                    tile(t, std::false_type());
                    tile(t + 1, std::true_type());
                }
                if (PAIRED && t + 1 < nt) {
                    tile(t, std::false_type());
                    t++;
                    __builtin_amdgcn_sched_barrier(0);
                    minima(0, t, std::true_type());
                    minima(1, t, std::true_type());
                } else {
                    __builtin_amdgcn_sched_barrier(0);
                    minima(0, t, std::false_type());
                    minima(1, t, std::false_type());
#pragma unroll
                    for (int s = 0; s < 2; s++) second[s] = PAIRED ? minimum(second[s], runner[s]) : second[s];
                }
            }
            // ---- the two halves of the wave hold different cells of the same rows; one exchange gives lane
            // half h both cells of the rows of set h, which it then decides
            float b, gap;
            int h_of;
            {
                const auto eb = __builtin_amdgcn_permlane32_swap(__float_as_uint(best[0]), __float_as_uint(best[1]),
                                                                 false, false);
                const auto es = __builtin_amdgcn_permlane32_swap(__float_as_uint(second[0]), __float_as_uint(second[1]),
                                                                 false, false);
                const float b0 = __uint_as_float(eb[0]), b1 = __uint_as_float(eb[1]);
                b = minimum(b0, b1);
                gap = minimum(minimum(__builtin_elementwise_maximum(b0, b1), __uint_as_float(es[0])),
                              __uint_as_float(es[1])) - b;
                h_of = b0 <= b1 ? 0 : 1;
            }
            const uint32_t cell = __float_as_uint(b) & a.cell_mask;
            bool open = !(gap > margin);  // the rule has to look at all entries
            // ---- the cell's 8 entries in fp32, again with the second best; rows too close to call join
            // the open ones
            {
                // the cell's entries are those from 16 * its number + 4h on, 4 of them and 4 from 8 further on
                const uint32_t c0 = open ? 0u : cell, h4 = open ? 0u : 4u * (uint32_t)h_of, e0 = c0 * 16u + h4;
                const float *near_ent = s_ent + __umul24(c0, GROUPS4) + __umul24(h4, GROUP / 4);
                float4 near_norm[2];
                if constexpr (ENT) {
                    near_norm[0] = *reinterpret_cast<const float4 *>(near_ent + 4 * WP);
                    near_norm[1] = *reinterpret_cast<const float4 *>(near_ent + 2 * GROUP + 4 * WP);
                }
                float b1 = 3e38f, b2 = 3e38f, key[2];
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    const int e = (int)e0 + (k & 3) + 8 * (k >> 2);
                    [[maybe_unused]] const float4 nn = near_norm[k >> 2];
                    [[maybe_unused]] const float norm = (k & 3) == 0 ? nn.x : (k & 3) == 1 ? nn.y : (k & 3) == 2 ? nn.z : nn.w;
                    float c[WP], rn, sc = 0.0f;
                    if constexpr (ENT) {
                        const float4 *src = reinterpret_cast<const float4 *>(near_ent + (k >> 2) * 2 * GROUP + (k & 3) * WP);
#pragma unroll
                        for (int i = 0; i < WP / 4; i++) {
                            const float4 v = src[i];
                            c[4 * i] = v.x; c[4 * i + 1] = v.y; c[4 * i + 2] = v.z; c[4 * i + 3] = v.w;
                        }
                        rn = norm;
                    } else {
                        entry(min(e, len - 1), c, rn);
                    }
                    if constexpr (COS) {
#pragma unroll
                        for (int d = 0; d < WP; d++) sc = fmaf(-xr[d], c[d], sc);
                        sc *= rn;
                    } else if constexpr (ENT) {
                        sc = norm;
#pragma unroll
                        for (int d = 0; d < WP; d++) sc = fmaf(-xr[d], c[d], sc);
                    } else {
#pragma unroll
                        for (int d = 0; d < WP; d++) sc = fmaf(c[d], fmaf(0.5f, c[d], -xr[d]), sc);
                    }
                    if ((!ENT || COS) && e >= len) sc = 3e38f;
                    key[k & 1] = __uint_as_float((__float_as_uint(sc) & ~7u) | (uint32_t)k);
                    if (k & 1) {
                        b2 = minimum(b2, __builtin_amdgcn_fmed3f(b1, key[0], key[1]));
                        b1 = minimum(minimum(b1, key[0]), key[1]);
                    }
                }
                const int k = (int)(__float_as_uint(b1) & 7u);
                open |= !(b2 - b1 > cell_margin);
                code = (int)e0 + (k & 3) + 8 * (k >> 2);
            }
            if (COS && zero) {  // all scores are zero: the first entry
                open = false;
                code = 0;
            }
            uint64_t todo = __ballot(open && valid);
            if constexpr (ENT) {
                if (__popcll(todo) > a.plain_rows) plain_left = kPlainStrips;
            } else {
                // (strips 0, 1 and 3, then every eighth)
                const bool look = strip < 4 ? strip != 2 : (strip & 7) == 7;
                strip++;
                if (look && __syncthreads_count(open && valid) > a.plain_rows * WAVES) {
                    plain = true;  // (the barrier: no wave reads the pieces any more)
                    float *dst = reinterpret_cast<float *>(s_frag);
                    for (int i = threadIdx.x; i < len * WP; i += TH) {
                        const int e = i / WP, d = i - e * WP;
                        dst[i] = d < w ? part_cb[(int64_t)e * w + d] : 0.0f;
                    }
                    __syncthreads();
                }
            }
            if (todo) {
                if ((ENT || plain) && __popcll(todo) >= a.lane_rows) {
                    search_all();
                    if (open) code = all_code;
                } else {
                    // two rows at a time, which halves the fetches of entries and has two reductions side by
                    // side, where there are registers for it (8 columns, entries in LDS, 4 waves a SIMD: the
                    // scores would lose 3 %)
                    constexpr int NR = WP == 16 || (WP == 8 && !ENT) ? 2 : 1;
                    while (todo) {
                        int j[NR];
                        float xj[NR][WP], bv[NR];
                        int bc[NR];
#pragma unroll
                        for (int n = 0; n < NR; n++) {
                            j[n] = todo ? __ffsll((unsigned long long)todo) - 1 : j[0];
                            todo &= todo - 1;
#pragma unroll
                            for (int d = 0; d < WP; d++)
                                xj[n][d] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(xr[d]), j[n]));
                            bv[n] = INFINITY;
                            bc[n] = 0x7FFFFFFF;
                        }
                        for (int e = lane; e < len; e += 64) {
                            float c[WP], rn;
                            entry(e, c, rn);
#pragma unroll
                            for (int n = 0; n < NR; n++) {
                                const float v = rule_value<WP, METRIC>(xj[n], c, rn);
                                if (v < bv[n]) { bv[n] = v; bc[n] = e; }
                            }
                        }
#pragma unroll
                        for (int n = 0; n < NR; n++) {
#pragma unroll
                            for (int o = 32; o > 0; o >>= 1) {
                                const float ov = __shfl_xor(bv[n], o);
                                const int oc = __shfl_xor(bc[n], o);
                                if (ov < bv[n] || (ov == bv[n] && oc < bc[n])) { bv[n] = ov; bc[n] = oc; }
                            }
                            if (lane == j[n]) code = bc[n] == 0x7FFFFFFF ? 0 : bc[n];
                        }
                    }
                }
            }
            }  // !plain
            if constexpr (TRAIN) {
                if (valid) {
                    float c[WP], rn;
                    entry(code, c, rn);
                    dsum += rule_value<WP, BIFEAT_VQ_L2>(xr, c, rn);
#pragma unroll
                    for (int d = 0; d < WP; d++)
                        if (d < w) unsafeAtomicAdd(&s_sum[d * len + code], (double)xr[d]);
                    atomicAdd(&s_cnt[code], 1u);
                }
            } else {
                // the next rows have arrived by now; waiting for them here keeps that wait from covering
                // the stores below (loads and stores of a wave complete in one order)
#pragma unroll
                for (int d = 0; d < WP; d++) asm volatile("" : "+v"(xn[d]));
                if (valid) {
                    if (a.cbytes == 1) *out = (uint8_t)code;
                    else *reinterpret_cast<uint16_t *>(out) = (uint16_t)code;
                    if (part == 0)
                        for (int64_t k = (int64_t)a.P * a.cbytes; k < a.rb; k++) out[k] = 0;  // padding
                }
                out += ROWS * a.rb;
            }
        }
        if constexpr (TRAIN) {
            const int this_set = set;
            set += a.sub > 1 ? a.sets : a.ny;
            if (a.one_set && set < a.sets) continue;  // (all sets' sums together)
            __syncthreads();
            const int64_t to = (a.one_set ? 0 : ((int64_t)this_set * a.sub + sub) * a.P) + part;
            float *sums = static_cast<float *>(a.sums) + to * len * w;
            uint32_t *counts = a.counts + to * len;
            if (a.one_set) {
                for (int i = threadIdx.x; i < len * w; i += TH)
                    if (s_sum[i] != 0.0) unsafeAtomicAdd(&sums[i], (float)s_sum[i]);
                for (int i = threadIdx.x; i < len; i += TH)
                    if (s_cnt[i]) atomicAdd(&counts[i], s_cnt[i]);
            } else {
                if (a.sub > 1) {
                    double *wide = static_cast<double *>(a.sums) + to * len * w;
                    for (int i = threadIdx.x; i < len * w; i += TH) wide[i] = s_sum[i];
                } else {
                    for (int i = threadIdx.x; i < len * w; i += TH) sums[i] = (float)s_sum[i];
                }
                for (int i = threadIdx.x; i < len; i += TH) counts[i] = s_cnt[i];
            }
            if (set < a.sets) {  // (the same thread's as read above)
                for (int i = threadIdx.x; i < len * w; i += TH) s_sum[i] = 0.0;
                for (int i = threadIdx.x; i < len; i += TH) s_cnt[i] = 0u;
                __syncthreads();
            }
        }
    } while (TRAIN && set < a.sets);
    if constexpr (TRAIN) {
        if (!COS && dsum != dsum) dsum = INFINITY;  // (a row that is near to no entry)
        for (int o = 32; o > 0; o >>= 1) dsum += __shfl_xor(dsum, o);
        if (lane == 0) unsafeAtomicAdd(&s_dist, (double)dsum);
        __syncthreads();
        if (threadIdx.x == 0) {
            // (id, from the registers that a workgroup starts with: one less to keep)
            if (a.one_set) unsafeAtomicAdd(a.distortion, s_dist);
            else a.distortion[(blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3)] = s_dist;
        }
    }
}

// Bound on how far the difference of two scores can be from what the rule decides on, relative to
// M = |x|^2 + max|c|^2 (scaled; every |score| and half of every squared distance is at most M;
// cosine: M = |x||c|).  u = 2^-24.
//   pieces: x rounded towards zero twice (2^-20 of each column), c to nearest twice (2^-22), the
//     product of the low pieces left out (2^-10 . 2^-11); by Cauchy at most 7 . 2^-22 M/2 per score,
//     and what is lost below the smallest normal half (2^-14 of codebooks scaled to 2^10) at most
//     2^-20 M: 2^-19 M per score
//   sums: at most 32 products per 8 columns and the constant added in fp32, each addition to 2u M;
//     the constant itself (w + 2) u M and, in pieces, 2^-33 of it
//   the cell number in the low bits: 2^(bits - 23) M
//   the rule: distances (w + 2) u relative, i.e. (w + 2) u M per score
// twice that for two scores, and a quarter on top (in which |x|^2 from the high pieces, short of it by
// less than 2^-9 of itself, is covered).
float vq_margin(int w, int len) {
    const double u = ldexp(1.0, -24);
    const int groups = (w + 7) / 8, cell_bits = ilog2(2 * ((len + 31) / 32));
    const double score = ldexp(1.0, -19) + 2.0 * u * (32.0 * groups + 2.0) + ldexp(1.0, cell_bits - 23) +
                         2.0 * u * (w + 4.0);
    return (float)(1.25 * 2.0 * score);
}

// whether the entries lie so densely in `cols` columns of a part that most rows are open, see vq_nearest_takes
bool too_dense(int w, int len, int cols) {
    const double gap = pow((double)len, -2.0 / cols) * std::min(1.0, 2.0 / cols);
    return vq_margin(w, len) > 0.01 * gap;
}

// The same for the scores inside a cell: fp32 throughout, (w + 4) u M, and three low bits.
float vq_cell_margin(int w) {
    const double u = ldexp(1.0, -24);
    return (float)(1.25 * 2.0 * (2.0 * (w + 4.0) * u + ldexp(1.0, 3 - 23)));
}

size_t nearest_lds(const bifeat_params *p, int G, int NT, bool ent, bool train) {
    const int w = p->scheme.vq_width, len = p->scheme.vq_length;
    size_t n = (size_t)NT * tile_units(G, ent) * 16 + (norm_slot(G, ent) ? 16 : sizeof(float) * NT * 32);
    if (ent) n += sizeof(float) * (size_t)NT * 2 * groups4_floats(G);
    if (train) n += (size_t)len * (sizeof(double) * w + sizeof(uint32_t));
    return n;
}

// Entries in LDS next to their pieces when they fit; else the pieces alone, the rule reading its few
// entries from L2.
bool entries_in_lds(const bifeat_params *p, bool train) {
    const int G = (p->scheme.vq_width + 7) / 8, tiles = (p->scheme.vq_length + 31) / 32;
    const int64_t limit = kCuLds - 1024;
    return (int64_t)nearest_lds(p, G, tiles, true, train) <= limit;
}

// Rows of a wave that the scores leave open are searched by the rule two at a time, the lanes sharing
// the codebook, or, from `lane_rows` of 64 on, all in one pass over it; and from `plain_rows` on the
// scores do not pay at all.  The costs in vector instructions, fitted to how many open rows of 64 make the
// scores as dear as the rule for all (65 536 rows; us with none open, per share of 1 up to 0.2, all by the
// rule; that number measured, and by the fit):
//   96 x 256 x 8   142, 2300, 732: 18.0, 18.0    48 x 1000 x 8  213, 2860, 1570: 31.2, 31.4   16 x 1000 x 16  132, 1580, 933: 30.2, 32.1
//   48 x 256 x 16  112, 1420, 765: 27.6, 23.2    24 x 512 x 16  108, 1560, 776: 28.6, 28.9    32 x 256 x 24  111, 1590, 723: 24.8, 24.1
//   24 x 256 x 32  108, 1570, 755: 25.4, 24.6    24 x 64 x 32  68, 840, 218: 11.9, 14.6
//   without the entries in LDS: 8 x 2048 x 16  175, 2450, 946: 22.5, 20.0   8 x 1500 x 24  203, 3130, 1060: 17.7, 19.5
//   8 x 1000 x 32  250, 7600, 950: 6.1, 6.1 (entries of 128 bytes meet in the caches)   8 x 1500 x 21  413, 16 000, 1080: 3.4
// By cosine the rule costs a multiplication and an addition instead of three instructions: 0.8 to 0.95 of these.
inline double rule_cost(int len, int G) { return len * (3.0 * 8 * G + 3.0); }
inline double scores_cost(int len, int G, bool ent) { return (ent ? 3.6 : G == 4 ? 6.5 : 4.7) * len * G + 400.0; }
template <typename T>
void search_costs(VqNearestArgs<T> &a, int G, bool ent, bool cosine) {
    const double entry = 3.0 * 8 * G + 3.0, all = rule_cost(a.len, G);
    // each lane its own entry
    const double apart = ent ? (G == 1 ? 1.3 : G == 2 ? 1.45 : G == 3 ? 1.65 : 1.75) : !a.bvec ? 14.0 : a.w == 32 ? 7.4 : 2.5;
    const double one = (a.len + 63) / 64 * entry * apart + 170.0;
    const double scores = scores_cost(a.len, G, ent);
    a.lane_rows = (int)std::min(64.0, all / one);
    // (a wave that decides by itself keeps to it for 7 more strips: 5 rows, more than their number's spread, on top)
    a.plain_rows = (int)std::max(1.0, std::min(60.0, (cosine ? 0.88 : 1.0) * (all - scores) / one + (ent ? 5.0 : 0.0)));
}

template <typename T, int G, int METRIC, bool ENT, bool TRAIN, int TH>
bool launch_one(bifeat_params *p, VqNearestArgs<T> a, uint8_t *codes, size_t lds, hipStream_t s) {
    auto kern = vq_nearest_kernel<T, G, METRIC, ENT, TRAIN, TH>;
    // (the kernel's few static words count too)
    if (lds > 65536 - 64 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    // Workgroups per part: one to four times what the chip holds at once, as the slots that stay empty
    // and the staging of the codebook, about as long as a strip, cost least (24 x 270 x 32, all rows
    // open: 845 us with one workgroup a CU, 1022 with two rounds of two).  In training, where each also
    // writes its sums to memory, as deal_sets has it.
    const int64_t resident =
        256 * std::min<int64_t>(ENT ? nearest_waves(G, true, TH) * 256 / TH : 1, kCuLds / (int64_t)lds);
    int64_t ny = 0;
    [[maybe_unused]] double *const distortion = a.distortion;
    if constexpr (TRAIN) {
        RowSets r = row_sets(p, a.rows);
        deal_sets(r, a.rows, a.P, resident, TH);
        ny = r.groups;
        // the sets' sums; without room for them (a stream that is being captured) they add to
        // the handle's own block of one set (10 rounds on 65 536 rows, with workspace / so: 8 x 256 x 16
        // 530 / 500 us, 96 x 256 x 8 1690 / 1650; one workgroup per part 8790 and 6370)
        const int64_t books = (int64_t)a.P * a.len * a.w, ents = (int64_t)a.P * a.len;
        if (ensure_scratch(p, (size_t)round_bytes(p, r, a.P), s)) {
            a.sums = p->d_scratch;
            a.counts = (uint32_t *)(p->d_scratch + r.sets * r.sub * books * (r.sub > 1 ? 8 : 4));
            a.distortion = round_dists(p, r, p->d_scratch);
        } else {
            a.one_set = 1;
            a.sums = p->d_train;
            a.counts = (uint32_t *)(p->d_train + books);
            launch_vq_zero(p->d_train, books + ents, s);
        }
        a.strip_log2 = r.strip_log2;
        a.sets = r.sets;
        a.sub = r.sub;
        a.chunk = r.share;
    } else {
        // A last part of so few columns that most of its rows go by the rule (see too_dense) costs as many times the
        // others and gets as many times their workgroups: dealt evenly, 100 000 half-precision rows of 601 columns by 8,
        // 256 entries, took 588 us, 202 so (608 columns: 160); 65 536 of 129 by 16 136, 62; of 769 by 16, 2048 entries, 5990, 1490.
        const int rest = (int)(p->D % a.w);
        const double last = !rest || !too_dense(a.w, a.len, rest) ? 1.0
                            : (METRIC == BIFEAT_VQ_COSINE ? 0.88 : 1.0) * rule_cost(a.len, G) / scores_cost(a.len, G, ENT);
        const int64_t strips = (a.rows + TH - 1) / TH;
        int64_t ny_last = 0;
        double least = 0.0;
        for (int m = 1; m <= 4; m++) {
            const int64_t n = (int64_t)(m * resident / (a.P - 1 + last));
            if (n < 1) continue;
            const int64_t n_last = last > 1.0 ? std::max(n, m * resident - n * (a.P - 1)) : n;
            const double rows_long = m * (std::max(1.0 / n, last / n_last) * a.rows + 0.8 * TH);
            if (least == 0.0 || rows_long < least) { least = rows_long; ny = n; ny_last = n_last; }
        }
        // (whole strips instead would leave the chip waiting for the workgroups with one more)
        auto deal = [&](int64_t &n, int64_t &chunk) {
            n = std::min(std::max<int64_t>(n, 1), strips);
            chunk = ((a.rows + n - 1) / n + 63) / 64 * 64;
            n = (a.rows + chunk - 1) / chunk;
        };
        deal(ny, a.chunk);
        deal(ny_last, a.last_chunk);
        a.more = (int)std::max<int64_t>(0, ny_last - ny);
    }
    a.ny = (int)ny;
    search_costs(a, G, ENT, METRIC == BIFEAT_VQ_COSINE);
    const int64_t blocks = ((int64_t)a.P * ny + a.more + 7) / 8 * 8;
    kern<<<(unsigned)blocks, TH, lds, s>>>(a, p->d_cb, codes);
    if constexpr (TRAIN)
        launch_vq_means(p, a.sums, a.counts, a.one_set ? 1 : a.sets, a.one_set ? 1 : a.sub,
                        a.one_set ? nullptr : a.distortion, a.P * a.ny, distortion, s);
    return true;
}

template <typename T, int G, int METRIC>
bool launch_metric(bifeat_params *p, VqNearestArgs<T> a, uint8_t *codes, hipStream_t s) {
    const bool train = codes == nullptr;
    const int tiles = (a.len + 31) / 32;
    const bool ent = entries_in_lds(p, train);
    a.NT = tiles;
    const size_t lds = nearest_lds(p, G, a.NT, ent, train);
    if (!ent) return train ? false : launch_one<T, G, METRIC, false, false, 512>(p, a, codes, lds, s);
#define BF_VNL(TH) (train ? launch_one<T, G, METRIC, true, true, TH>(p, a, codes, lds, s) \
                          : launch_one<T, G, METRIC, true, false, TH>(p, a, codes, lds, s))
    // Workgroups of 256 threads while a CU holds three or more.  Larger codebooks would leave it with few
    // waves, so they are shared by as many as the registers allow: 65 536 rows of 96 x 1000 x 8 459 us (512
    // threads that read the entries from L2: 726), 48 x 512 x 16 207 (358), 24 x 270 x 32 124 (447); training
    // 96 x 1000 x 8 4680 us (search and sums apart 5050).  9 to 16 columns: with three waves a SIMD in mind the
    // plain search spills, which workgroups of 512 do not have (48 x 512 x 16 244 in two of 256).
    // (the kernel's few static words count too)
    const int64_t fit = kCuLds / ((int64_t)lds + 64);
    // (training at two a CU: as many sets, with one codebook for each)
    if (fit >= 3 || (train && fit == 2 && G >= 2)) return BF_VNL(256);
    if constexpr (G == 1) return fit == 2 ? BF_VNL(512) : BF_VNL(1024);
    else return BF_VNL(512);
#undef BF_VNL
}

template <typename T, int G>
bool launch_groups(bifeat_params *p, VqNearestArgs<T> a, uint8_t *codes, hipStream_t s) {
    const int cell_bits = ilog2(2 * ((a.len + 31) / 32));
    a.margin = vq_margin(a.w, a.len);
    a.cell_margin = vq_cell_margin(a.w);
    a.cell_mask = (1u << cell_bits) - 1u;
    return p->scheme.vq_metric == BIFEAT_VQ_COSINE ? launch_metric<T, G, BIFEAT_VQ_COSINE>(p, a, codes, s)
                                                   : launch_metric<T, G, BIFEAT_VQ_L2>(p, a, codes, s);
}

// codes == nullptr: training
template <typename T>
bool launch_nearest(bifeat_params *p, const T *x, int64_t rows, uint8_t *codes, int64_t rb, int64_t pb,
                    double *distortion, hipStream_t s) {
    const int w = p->scheme.vq_width, len = p->scheme.vq_length;
    if (!vq_nearest_takes(p, !codes, rows)) return false;
    VqNearestArgs<T> a{};
    a.x = x;
    a.rows = rows;
    a.D = (int)p->D;
    a.w = w;
    a.len = len;
    a.P = p->P;
    a.cbytes = p->cbytes;
    a.bvec = w % 4 == 0;
    a.rnorm = p->d_rnorm;
    a.rb = rb;
    a.pb = pb;
    a.distortion = distortion;
    switch ((w + 7) / 8) {
        case 1: return launch_groups<T, 1>(p, a, codes, s);
        case 2: return launch_groups<T, 2>(p, a, codes, s);
        case 3: return launch_groups<T, 3>(p, a, codes, s);
        default: return launch_groups<T, 4>(p, a, codes, s);
    }
}

}  // namespace

template <typename T>
bool launch_vq_nearest_codes(bifeat_params *p, const T *x, int64_t rows, uint8_t *codes, int64_t rb, int64_t pb,
                             hipStream_t s) {
    return launch_nearest<T>(p, x, rows, codes, rb, pb, nullptr, s);
}

template <typename T>
bool launch_vq_nearest_round(bifeat_params *p, const T *x, int64_t rows, double *distortion, hipStream_t s) {
    return launch_nearest<T>(p, x, rows, nullptr, 0, 0, distortion, s);
}

#define BF_VN(T)                                                                                              \
    template bool launch_vq_nearest_codes<T>(bifeat_params *, const T *, int64_t, uint8_t *, int64_t, int64_t,       \
                                             hipStream_t);                                                     \
    template bool launch_vq_nearest_round<T>(bifeat_params *, const T *, int64_t, double *, hipStream_t);

}  // namespace bf
