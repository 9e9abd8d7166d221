// Codebook training for the vector codes (paper Sec. 3.2: k-means per part;
// Appendix D: on a uniform row sample, and names the GPU as the place to run it).
//
// Lloyd rounds on a sample chunk resident in GPU memory: initial entries = the
// sample's first `length` rows (per part); each round assigns every sample
// sub-vector to its nearest entry (the same fp32 rule as the encoder, so a
// trained codebook encodes exactly as it was fitted), accumulates per-entry
// sums and counts and replaces each non-empty entry by the mean of its members
// (an entry without members keeps its value).  Sums are 64-bit LDS atomics, rounded to 32 bits set by
// set (RowSets): the same sample gives the same codebook on every path that has room for its sums, up
// to a sum that lies within 2^-53 of an edge between two 32-bit values.  The plain fused kernel, and
// sums that find no room, depend on the order of additions in the last bits.
// Three forms:
// - codebooks that the matrix-core search takes and that fit LDS next to their sums: search and
//   sums in one kernel (vq_nearest.hip; 96 x 256 x 8 cosine, 10 rounds on 65 536 rows: 1760 us,
//   apart 2090; 96 x 512 x 8 2590 and 3070);
// - everything else that the plain fused kernel cannot do (cosine metric, two-byte codes) or
//   does badly (codes_pay below) runs the encoder's own kernel into a scratch code array and
//   adds up from that, in LDS and per workgroup;
// - the plain fused kernel (sums in LDS in 32 bits, then global atomics) for the rest, and
//   for those of the second form's codebooks that it can do where a stream under capture
//   leaves no room for the codes.
#include "common.hpp"
#include "vq_nearest.hpp"

#include <algorithm>

namespace bf {

namespace {

// cb[p][c][d] = x[c][p*w + d] for c < len (columns past D read as 0)
template <typename T>
__global__ void vq_init_kernel(const T *__restrict__ x, int D, int w, int len, int P,
                               float *__restrict__ cb) {
    const int64_t n = (int64_t)P * len * w;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int d = (int)(i % w), c = (int)((i / w) % len), p = (int)(i / ((int64_t)w * len));
        const int col = p * w + d;
        cb[i] = col < D ? load1(x + (int64_t)c * D + col) : 0.0f;
    }
}

__global__ void vq_zero_kernel(float *__restrict__ a, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        a[i] = 0.0f;
}

// one workgroup = one part x a strip of sample rows
template <typename T, int W>
__global__ __launch_bounds__(kThreads) void vq_lloyd_accumulate_kernel(
    const T *__restrict__ x, int64_t rows, int D, int w_rt, int len, const float *__restrict__ cb,
    float *__restrict__ sums, float *__restrict__ counts, double *__restrict__ distortion) {
    extern __shared__ float sm[];
    const int w = W > 0 ? W : w_rt;
    float *s_cb = sm, *s_sum = sm + len * w, *s_cnt = s_sum + len * w;
    const int p = blockIdx.x;
    for (int i = threadIdx.x; i < len * w; i += kThreads) {
        s_cb[i] = cb[(int64_t)p * len * w + i];
        s_sum[i] = 0.0f;
    }
    for (int i = threadIdx.x; i < len; i += kThreads) s_cnt[i] = 0.0f;
    __syncthreads();
    float dsum = 0.0f;
    for (int64_t r = (int64_t)blockIdx.y * kThreads + threadIdx.x; r < rows;
         r += (int64_t)gridDim.y * kThreads) {
        const T *src = x + r * D + (int64_t)p * w;
        int best = 0;
        float bestd = INFINITY;
        if constexpr (W > 0) {
            float sub[W];
#pragma unroll
            for (int d = 0; d < W; d++) sub[d] = (p * W + d < D) ? load1(src + d) : 0.0f;
            for (int c = 0; c < len; c++) {
                float dist = 0.0f;
#pragma unroll
                for (int d = 0; d < W; d++) {
                    const float diff = __fsub_rn(sub[d], s_cb[c * W + d]);
                    dist = __fadd_rn(dist, __fmul_rn(diff, diff));
                }
                if (dist < bestd) { bestd = dist; best = c; }
            }
#pragma unroll
            for (int d = 0; d < W; d++) atomicAdd(&s_sum[best * W + d], sub[d]);
        } else {
            for (int c = 0; c < len; c++) {
                float dist = 0.0f;
                for (int d = 0; d < w; d++) {
                    const float xv = (p * w + d < D) ? load1(src + d) : 0.0f;
                    const float diff = __fsub_rn(xv, s_cb[c * w + d]);
                    dist = __fadd_rn(dist, __fmul_rn(diff, diff));
                }
                if (dist < bestd) { bestd = dist; best = c; }
            }
            for (int d = 0; d < w; d++)
                atomicAdd(&s_sum[best * w + d], (p * w + d < D) ? load1(src + d) : 0.0f);
        }
        atomicAdd(&s_cnt[best], 1.0f);
        dsum += bestd;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < len * w; i += kThreads)
        if (s_sum[i] != 0.0f) atomicAdd(&sums[(int64_t)p * len * w + i], s_sum[i]);
    for (int i = threadIdx.x; i < len; i += kThreads)
        if (s_cnt[i] != 0.0f) atomicAdd(&counts[(int64_t)p * len + i], s_cnt[i]);
    for (int o = 32; o > 0; o >>= 1) dsum += __shfl_xor(dsum, o);
    if ((threadIdx.x & 63) == 0) unsafeAtomicAdd(distortion, (double)dsum);
}

__global__ void vq_lloyd_update_kernel(float *__restrict__ cb, const float *__restrict__ sums,
                                       const float *__restrict__ counts, int w, int64_t n,
                                       const double *__restrict__ distortion, int rounds, double *host) {
    if (host && blockIdx.x == 0 && (int)threadIdx.x < rounds) host[threadIdx.x] = distortion[threadIdx.x];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const float cnt = counts[i / w];
        if (cnt > 0.0f) cb[i] = sums[i] / cnt;
    }
}

template <typename T>
void lloyd_round(bifeat_params *p, const T *x, int64_t rows, double *dist_slot, hipStream_t s) {
    // codebooks that the matrix-core search leaves and codes do not pay for, or have no workspace for
    const int w = p->scheme.vq_width, len = p->scheme.vq_length, P = p->P;
    const int64_t n = (int64_t)P * len * w;
    float *sums = p->d_train, *counts = p->d_train + n;
    vq_zero_kernel<<<256, 256, 0, s>>>(p->d_train, n + (int64_t)P * len);
    int64_t strips = (rows + kThreads * 8 - 1) / (kThreads * 8);  // ~8 rows per thread
    if (strips < 1) strips = 1;
    if (strips > 1024) strips = 1024;
    dim3 grid((unsigned)P, (unsigned)strips);
    const size_t shm = sizeof(float) * ((size_t)2 * len * w + len);
#define BF_LL(W) \
    vq_lloyd_accumulate_kernel<T, W><<<grid, kThreads, shm, s>>>(x, rows, (int)p->D, w, len, p->d_cb, sums, counts, dist_slot)
    switch (w) {
        case 1: BF_LL(1); break;
        case 2: BF_LL(2); break;
        case 4: BF_LL(4); break;
        case 8: BF_LL(8); break;
        case 16: BF_LL(16); break;
        default: BF_LL(0); break;
    }
#undef BF_LL
    const int k = (int)(dist_slot - p->d_dist);
    vq_lloyd_update_kernel<<<256, 256, 0, s>>>(p->d_cb, sums, counts, w, n, p->d_dist, k + 1, last_round(p, k));
}

// rnorm[i] = fp32(1 / sqrt(sum_d C_id^2)), 0 for an all-zero entry; sum and root in fp64
__global__ void vq_rnorm_kernel(const float *__restrict__ cb, int64_t entries, int w,
                                float *__restrict__ rnorm) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < entries;
         i += (int64_t)gridDim.x * blockDim.x) {
        double ss = 0.0;
        for (int d = 0; d < w; d++) ss += (double)cb[i * w + d] * (double)cb[i * w + d];
        rnorm[i] = ss > 0.0 ? (float)(1.0 / sqrt(ss)) : 0.0f;
    }
}

// Sums, counts and squared distance from the codes, one part's after the other.  A workgroup takes
// one part, as many of its columns (the count is one more) as LDS holds sums for - 64-bit ones, see
// vq_nearest.hip - and the rows of a set, of several one after the other, or of part of one, and writes
// each one's sums to the workspace; or adds them to the one (zeroed) set there is room for.
// What bounds it: the LDS adds (22 cycles a wave, 36 us for 65 536 rows of 96 x 8 columns) and reading
// the sample once more (40 us).  For that 4 columns are loaded at a time (VEC) and lanes share a row
// (a load of one lane per row touches 64 lines), workgroups of the same rows run at the same time on one
// XCD (four parts of 8 columns share a line), and a wave's codes are consecutive.  A round's sums of
// that shape: 68 us; one lane per row 89; with 4-byte loads, codes row by row and the parts dealt over
// the XCDs 475.
constexpr int kAccThreads = 1024;
constexpr int64_t kAccLds = 145 * 1024;
constexpr int kAccRows = 2;
constexpr int64_t kMaxSumsBytes = (int64_t)256 << 20;
// from one column's sums to the next: odd, so that lanes that add columns of one row meet different banks
__host__ __device__ constexpr int acc_stride(int len) { return len | 1; }

template <typename T, typename CODE, bool VEC>
__global__ __launch_bounds__(kAccThreads) void vq_accumulate_codes_kernel(
    const T *__restrict__ x, int64_t rows, int D, int w, int len, int P, const CODE *__restrict__ codes,
    const float *__restrict__ cb, int DG, int more, int groups, RowSets r, int lanes, int one_set, int l2,
    void *__restrict__ all_sums, uint32_t *__restrict__ counts, double *__restrict__ distortion) {
    extern __shared__ double s_acc[];  // [columns][acc_stride]
    const int ls = acc_stride(len);
    __shared__ double s_dist;
    // workgroups are dealt to the XCDs in turn: consecutive logical ids belong on one XCD
    const int id = (int)((blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3)), TH = blockDim.x;
    if (id >= groups * P * r.groups) return;
    const int grp = id % groups, p = id / groups % P, by = id / (groups * P), sub = by % r.sub;
    const int c0 = grp * DG, nc = min(DG + (grp == groups - 1 ? more : 0), w + 1 - c0);  // column w counts
    const int nd = min(nc, w - c0);
    for (int i = threadIdx.x; i < nc * ls; i += TH) s_acc[i] = 0.0;
    if (threadIdx.x == 0) s_dist = 0.0;
    __syncthreads();
    float dsum = 0.0f;
    const CODE *part_codes = codes + p * rows;
    const int left = D - (p * w + c0);  // columns that the table has
    auto add = [&](double *acc, int j, float xv, float ev) {
        unsafeAtomicAdd(acc + j * ls, (double)xv);
        const float diff = xv - ev;
        dsum += diff * diff;
    };
    // (rows are counted within the set)
    for (int set = by / r.sub, next; set < r.sets; set = next) {
        next = set + (r.sub > 1 ? r.sets : r.groups);
        const int64_t begin = sub * r.share, end = min(set_rows(set, r.sets, r.strip_log2, rows), begin + r.share);
        if constexpr (VEC) {
            // (rows that begin anywhere; `left` ends in the middle of a four in the last part only)
            // `lanes` lanes (a power of two that divides the fours of columns) share a row: fewer lines an
            // instruction; a lane has kAccRows rows in flight
            const int lq = threadIdx.x & (lanes - 1), at = threadIdx.x / lanes, step = TH / lanes;
            for (int64_t i = begin + at; i < end; i += (int64_t)step * kAccRows) {
                int code[kAccRows];
                int64_t row[kAccRows];
#pragma unroll
                for (int k = 0; k < kAccRows; k++) {
                    row[k] = set_row(set, r.sets, r.strip_log2, i + k * step);
                    code[k] = i + k * step < end ? part_codes[row[k]] : -1;
                }
                for (int j = 4 * lq; j < nd; j += 4 * lanes) {
                    float4 v[kAccRows], e[kAccRows];
#pragma unroll
                    for (int k = 0; k < kAccRows; k++) {
                        v[k] = e[k] = make_float4(0.f, 0.f, 0.f, 0.f);
                        if (code[k] < 0) continue;
                        const T *src = x + row[k] * D + (int64_t)p * w + c0 + j;
                        if (j + 4 <= left) {
                            v[k] = load4_any(src);
                        } else if (j < left) {
                            v[k].x = load1(src);
                            if (j + 1 < left) v[k].y = load1(src + 1);
                            if (j + 2 < left) v[k].z = load1(src + 2);
                        }
                        e[k] = load4(cb + ((int64_t)p * len + code[k]) * w + c0 + j);
                    }
#pragma unroll
                    for (int k = 0; k < kAccRows; k++) {
                        if (code[k] < 0) continue;
                        double *acc = s_acc + code[k];
                        add(acc, j, v[k].x, e[k].x);
                        add(acc, j + 1, v[k].y, e[k].y);
                        add(acc, j + 2, v[k].z, e[k].z);
                        add(acc, j + 3, v[k].w, e[k].w);
                    }
                }
                if (nc > nd && lq == 0) {
#pragma unroll
                    for (int k = 0; k < kAccRows; k++)
                        if (code[k] >= 0) unsafeAtomicAdd(s_acc + code[k] + nd * ls, 1.0);
                }
            }
        } else {
            for (int64_t i = begin + threadIdx.x; i < end; i += TH) {
                const int64_t row = set_row(set, r.sets, r.strip_log2, i);
                const int code = part_codes[row];
                const T *src = x + row * D + (int64_t)p * w + c0;
                const float *ent = cb + ((int64_t)p * len + code) * w + c0;
                double *acc = s_acc + code;
#pragma unroll 4
                for (int j = 0; j < nd; j++) add(acc, j, j < left ? load1(src + j) : 0.0f, ent[j]);
                if (nc > nd) unsafeAtomicAdd(acc + nd * ls, 1.0);
            }
        }
        if (one_set && next < r.sets) continue;  // (all sets' sums together)
        __syncthreads();
        for (int i = threadIdx.x; i < nc * len; i += TH) {
            const int j = i / len, e = i - j * len, d = c0 + j;
            const double sum = s_acc[j * ls + e];
            s_acc[j * ls + e] = 0.0;
            float *sums = static_cast<float *>(all_sums);
            const int64_t slot = (int64_t)set * r.sub + sub;
            if (one_set) {
                if (sum == 0.0) continue;
                if (d < w) unsafeAtomicAdd(&sums[((int64_t)p * w + d) * len + e], (float)sum);
                else atomicAdd(&counts[(int64_t)p * len + e], (uint32_t)sum);
            } else if (d < w) {
                const int64_t to = ((slot * P + p) * w + d) * len + e;
                if (r.sub > 1) static_cast<double *>(all_sums)[to] = sum;
                else sums[to] = (float)sum;
            } else {
                counts[(slot * P + p) * len + e] = (uint32_t)sum;
            }
        }
        __syncthreads();
    }
    if (l2 && dsum != dsum) dsum = INFINITY;  // (a row that is near to no entry)
    for (int o = 32; o > 0; o >>= 1) dsum += __shfl_xor(dsum, o);
    if ((threadIdx.x & 63) == 0) unsafeAtomicAdd(&s_dist, (double)dsum);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (one_set) unsafeAtomicAdd(distortion, s_dist);
        else distortion[(blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3)] = s_dist;  // [id]
    }
}

// The generic round's workspace: the codes, then the workgroups' sums.
struct GenericPlan {
    int DG, more, groups;            // columns a group, 1: the last one counts on top of them
    int threads;
    RowSets sets;
    int64_t codes_bytes, sums_bytes;  // codes (rounded up), sums, counts and distances of every workgroup
};

GenericPlan generic_plan(const bifeat_params *p, int64_t rows) {
    const int w = p->scheme.vq_width, len = p->scheme.vq_length;
    GenericPlan g;
    g.DG = (int)(kAccLds / (8 * acc_stride(len)));  // at least one: 16384 entries take 128 KB
    g.more = 0;
    if (w % 4 == 0 && g.DG > 4) {  // whole fours of columns, for wide loads
        g.more = 1;
        g.DG = std::min((g.DG - 1) / 4 * 4, w);
        g.groups = (w + g.DG - 1) / g.DG;
        g.DG = (w / 4 + g.groups - 1) / g.groups * 4;
    } else {
        if (g.DG > w + 1) g.DG = w + 1;
        g.groups = (w + g.DG) / g.DG;
        g.DG = (w + g.groups) / g.groups;
    }
    // smaller workgroups where a sample is too short to fill the chip with large ones, unless a
    // workgroup's sums outnumber its rows then (3000 rows of 8 x 2048 x 16: 730 us against 930) or there
    // are few columns to add (4096 rows of 24 x 64 x 4 cosine: 233 us against 262)
    const int64_t lds = (int64_t)8 * (g.DG + g.more) * acc_stride(len), cols = (int64_t)p->P * g.groups;
    g.threads = kAccThreads;
    while (w >= 8 && g.threads > 256 && g.threads / 2 >= len && cols * ((rows + g.threads - 1) / g.threads) < 512) g.threads /= 2;
    g.codes_bytes = (rows * p->P * p->cbytes + 255) / 256 * 256;
    g.sets = row_sets(p, rows);
    deal_sets(g.sets, rows, cols, 256 * std::min<int64_t>(2, 160 * 1024 / (lds + 64)), g.threads);
    if (g.sets.sub > 1 && sums_bytes(p, g.sets) > kMaxSumsBytes) g.sets = row_sets(p, rows);
    g.sums_bytes = round_bytes(p, g.sets, cols);
    return g;
}

// Whether a codebook that the plain fused kernel can train, and the matrix-core search does not take,
// goes through codes.  The fused kernel reads the sample once a round and is bound by its LDS float
// adds; the other way reads twice and adds in 64 bits at a ninth of the cost.  10 rounds, us, fused /
// codes: 65 536 x 24 x 64 x 1 657 / 422, 16 384 x 96 x 250 x 2 1250 / 1100, 65 536 x 6 x 16 x 4 274 / 277.
// Of one or two columns there is little to add, and at millions of parts with more than 64 entries the
// search is all that counts, which reads the sample as it lies in both (65 536 x 96 x 256 x 1 2390 / 2670).
bool codes_pay(const bifeat_params *p, int64_t rows) {
    return p->scheme.vq_width > 2 || p->scheme.vq_length <= 64 || rows * p->P < (1 << 22);
}

template <typename T, typename CODE, bool VEC>
bool accumulate_codes(bifeat_params *p, const T *x, int64_t rows, const GenericPlan &g, bool one_set, void *sums,
                      uint32_t *counts, double *distortion, hipStream_t s) {
    const size_t shm = sizeof(double) * (size_t)(g.DG + g.more) * acc_stride(p->scheme.vq_length);
    auto kern = vq_accumulate_codes_kernel<T, CODE, VEC>;
    if (shm > 65536 - 64 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)shm) != hipSuccess)
        return false;
    const int blocks = (g.groups * p->P * g.sets.groups + 7) / 8 * 8;
    int lanes = 1;
    while (VEC && lanes < 16 && g.DG % (8 * lanes) == 0) lanes *= 2;
    kern<<<(unsigned)blocks, g.threads, shm, s>>>(
        x, rows, (int)p->D, p->scheme.vq_width, p->scheme.vq_length, p->P, (const CODE *)p->d_scratch, p->d_cb, g.DG,
        g.more, g.groups, g.sets, lanes, one_set, p->scheme.vq_metric == BIFEAT_VQ_L2, sums, counts, distortion);
    return true;
}

template <typename T>
hipError_t lloyd_round_generic(bifeat_params *p, const T *x, int64_t rows, double *dist_slot, hipStream_t s) {
    const int w = p->scheme.vq_width, len = p->scheme.vq_length, P = p->P;
    const int64_t books = (int64_t)P * len * w;
    const GenericPlan g = generic_plan(p, rows);
    // without room for every workgroup's sums (a stream under capture) they add to the handle's own
    // block of one set (the codes' part of the workspace is there, see below): 8 x 2048 x 16 cosine,
    // 10 rounds 1960 us so, with workspace 2020; one workgroup per part and group of columns 8690
    const bool all = (int64_t)p->scratch_bytes >= g.codes_bytes + g.sums_bytes;
    const int sets = all ? g.sets.sets : 1, sub = all ? g.sets.sub : 1;
    uint8_t *sums = all ? p->d_scratch + g.codes_bytes : (uint8_t *)p->d_train;
    uint32_t *counts = (uint32_t *)(sums + sets * sub * books * (sub > 1 ? 8 : 4));
    double *dists = all ? round_dists(p, g.sets, sums) : nullptr, *distortion = all ? dists : dist_slot;
    if (!all) launch_vq_zero(p->d_train, books + (int64_t)P * len, s);
    if (p->scheme.vq_metric == BIFEAT_VQ_COSINE) launch_vq_rnorm(p, s);
    launch_vq_assign_parts(p, x, rows, p->d_scratch, s);
    // 4 columns at a time: whole fours of parts and of groups
    const bool vec = g.DG % 4 == 0 && w % 4 == 0;
    const bool ok = p->cbytes == 1
                        ? (vec ? accumulate_codes<T, uint8_t, true>(p, x, rows, g, !all, sums, counts, distortion, s)
                               : accumulate_codes<T, uint8_t, false>(p, x, rows, g, !all, sums, counts, distortion, s))
                        : (vec ? accumulate_codes<T, uint16_t, true>(p, x, rows, g, !all, sums, counts, distortion, s)
                               : accumulate_codes<T, uint16_t, false>(p, x, rows, g, !all, sums, counts, distortion, s));
    if (!ok) return hipGetLastError();
    launch_vq_means(p, sums, counts, sets, sub, dists, g.groups * P * g.sets.groups, dist_slot, s);
    return hipSuccess;
}

}  // namespace

// The handle's workspace (transposed codes of a vector-code gather, code array of the generic
// Lloyd rounds).  It only grows, and a buffer that was handed to kernels is never freed before
// the handle is destroyed: work still in flight, and HIP graphs captured from earlier calls,
// keep a valid address.  While `s` is being captured into a graph nothing is allocated: the
// request then fails unless a call (or bifeat_reserve) at least as large ran before.
bool ensure_scratch(bifeat_params *p, size_t bytes, hipStream_t s) {
    if (p->scratch_bytes >= bytes) return true;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    if (cap != hipStreamCaptureStatusNone) return false;
    void *q = nullptr;
    const size_t want = bytes + bytes / 4;
    if (hipMalloc(&q, want) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    if (p->d_scratch) p->retired.push_back(p->d_scratch);
    p->d_scratch = (uint8_t *)q;
    p->scratch_bytes = want;
    return true;
}

// rows of the largest set
static int64_t largest_set(const RowSets &r, int64_t rows) {
    const int64_t strips = (rows + (1 << r.strip_log2) - 1) >> r.strip_log2;
    return (strips + r.sets - 1) / r.sets << r.strip_log2;
}

// Sets of strips of 256 rows, as many as the chip holds workgroups of the search and its sums, for the Euclidean
// one-byte codebooks of 512 values or more, within 64 KB, that the matrix-core search trains; else of 1024 rows, as
// many as give two workgroups of the sums from codes a CU.
RowSets row_sets(const bifeat_params *p, int64_t rows) {
    const int64_t w = p->scheme.vq_width, len = p->scheme.vq_length;
    RowSets r{};
    int64_t sets;
    if (p->scheme.vq_metric == BIFEAT_VQ_L2 && p->cbytes == 1 && w * len >= 512 && 4 * len * (2 * w + 1) <= 65536 &&
        vq_nearest_takes(p, true, rows)) {
        const int64_t G = (w + 7) / 8, pairs = (len + 63) / 64;  // of tiles of 32 entries
        const int64_t lds = pairs * (2 * (1024 * G + 128) + 4 * (16 * (32 * G + 4) + 4)) + len * (8 * w + 4);
        r.strip_log2 = 8;
        sets = 256 * std::min<int64_t>(G == 1 ? 4 : G == 2 ? 3 : 2, 160 * 1024 / lds) / p->P;
    } else {
        const int64_t cols = std::min(144 * 1024 / (8 * len), w + 1);  // a workgroup's, one more counts
        r.strip_log2 = 10;
        sets = std::min(512 / (p->P * ((w + cols) / cols)), kMaxSumsBytes / (4 * p->P * len * (w + 1)));
    }
    r.sets = r.groups = (int)std::max<int64_t>(1, std::min(sets, (rows + (1 << r.strip_log2) - 1) >> r.strip_log2));
    r.sub = 1;
    r.share = largest_set(r, rows);
    return r;
}

// Several workgroups to a set while that many are missing; else one or several sets to a workgroup, as the rows of
// as many rounds of workgroups as it takes cost least, with staging a codebook and writing sums as long as 0.8
// and 0.4 rows a thread.
void deal_sets(RowSets &r, int64_t rows, int64_t cols, int64_t room, int threads) {
    const int64_t most = largest_set(r, rows);
    r.sub = (int)std::max<int64_t>(1, std::min(room / (cols * r.sets), (most + threads - 1) / threads));
    r.share = ((most + r.sub - 1) / r.sub + 63) / 64 * 64;
    r.groups = r.sets * r.sub;
    double least = 0.0;
    for (int m = 1; r.sub == 1 && m <= 8; m++) {
        const int64_t n = (r.sets + m - 1) / m, rounds = (n * cols + room - 1) / room;
        const double time = (double)rounds * (m * ((double)most + 0.4 * threads) + 0.8 * threads);
        if (least == 0.0 || time < least) { least = time; r.groups = (int)n; }
    }
}

void launch_vq_zero(float *a, int64_t n, hipStream_t s) {
    vq_zero_kernel<<<blocks_for(n, 1024), kThreads, 0, s>>>(a, n);
}

void launch_vq_rnorm(bifeat_params *p, hipStream_t s) {
    const int64_t entries = (int64_t)p->P * p->scheme.vq_length;
    vq_rnorm_kernel<<<blocks_for(entries), kThreads, 0, s>>>(p->d_cb, entries, p->scheme.vq_width,
                                                            p->d_rnorm);
}

// rounds Lloyd iterations over the sample chunk; init = true first seeds the
// codebooks from the chunk's first `length` rows.  d_dist[k] receives the summed
// squared distance of round k's assignment step.
hipError_t launch_vq_train(bifeat_params *p, const void *chunk, int dtype, int64_t rows, bool init,
                           int rounds, hipStream_t s) {
    const int w = p->scheme.vq_width, len = p->scheme.vq_length, P = p->P;
    const bool fused = p->scheme.vq_metric == BIFEAT_VQ_L2 && p->cbytes == 1 &&
                       sizeof(float) * ((size_t)2 * len * w + len) <= 65536;
    const GenericPlan g = generic_plan(p, rows);
    // (codes without the sums: see lloyd_round_generic)
    auto room_for_codes = [&] {
        return ensure_scratch(p, (size_t)(g.codes_bytes + g.sums_bytes), s) ||
               ensure_scratch(p, (size_t)rows * P * p->cbytes, s);
    };
    bool nearest = vq_nearest_takes(p, true, rows), through_codes = false;
    if (!nearest) {
        through_codes = fused ? codes_pay(p, rows) && ensure_scratch(p, (size_t)(g.codes_bytes + g.sums_bytes), s)
                              : room_for_codes();
        if (!fused && !through_codes) return hipErrorOutOfMemory;
    } else if (!fused && !vq_nearest_takes(p, true, 1)) {
        // A smaller sample of this codebook goes through codes and cannot do without them: a captured update of
        // one finds room for them after this one, as after any larger update.
        (void)ensure_scratch(p, (size_t)std::min(rows * P, kNearestManyParts) * p->cbytes, s);
    }
    if (init) {
        if (dtype == BIFEAT_F32)
            vq_init_kernel<float><<<256, 256, 0, s>>>((const float *)chunk, (int)p->D, w, len, P, p->d_cb);
        else
            vq_init_kernel<__half><<<256, 256, 0, s>>>((const __half *)chunk, (int)p->D, w, len, P, p->d_cb);
    }
    vq_zero_kernel<<<1, 128, 0, s>>>(reinterpret_cast<float *>(p->d_dist), 2 * rounds);
    auto round = [&](auto *x, double *dist) {
        if (nearest) {
            if (p->scheme.vq_metric == BIFEAT_VQ_COSINE) launch_vq_rnorm(p, s);
            if (launch_vq_nearest_round(p, x, rows, dist, s)) return hipSuccess;
            nearest = false;  // the runtime did not grant the LDS
            through_codes = !fused && room_for_codes();
            if (!fused && !through_codes) return hipErrorOutOfMemory;
        }
        if (through_codes) return lloyd_round_generic(p, x, rows, dist, s);
        lloyd_round(p, x, rows, dist, s);
        return hipSuccess;
    };
    for (int k = 0; k < rounds; k++) {
        const hipError_t e = dtype == BIFEAT_F32 ? round((const float *)chunk, p->d_dist + k)
                                                 : round((const __half *)chunk, p->d_dist + k);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

}  // namespace bf
