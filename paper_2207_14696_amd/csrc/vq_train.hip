// Codebook training for the vector codes (paper Sec. 3.2: k-means per part;
// Appendix D: on a uniform row sample, and names the GPU as the place to run it).
//
// Lloyd rounds on a sample chunk resident in GPU memory: initial entries = the
// sample's first `length` rows (per part); each round assigns every sample
// sub-vector to its nearest entry (the same fp32 rule as the encoder, so a
// trained codebook encodes exactly as it was fitted), accumulates per-entry
// sums and counts and replaces each non-empty entry by the mean of its members
// (an entry without members keeps its value).  Sums are added with atomics, so the result
// depends on the order of additions in the last bits; it is judged on distortion, not bit
// for bit.
// Three forms:
// - Euclidean one-byte codebooks that the matrix-core search takes: search and sums in one
//   kernel (vq_nearest.hip);
// - everything else that the plain fused kernel cannot do (cosine metric, two-byte codes) or
//   does badly (codes_pay below) runs the encoder's own kernel into a scratch code array and
//   adds up from that, in LDS and per workgroup;
// - the plain fused kernel (sums in LDS in 32 bits, then global atomics) for the rest, and
//   for those of the second form's codebooks that it can do where a stream under capture
//   leaves no room for the codes.
#include "common.hpp"
#include "vq_nearest.hpp"

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
                                       const float *__restrict__ counts, int w, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const float cnt = counts[i / w];
        if (cnt > 0.0f) cb[i] = sums[i] / cnt;
    }
}

template <typename T>
void lloyd_round(bifeat_params *p, const T *x, int64_t rows, double *dist_slot, hipStream_t s) {
    if (launch_vq_nearest_round<T>(p, x, rows, dist_slot, s)) return;
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
    vq_lloyd_update_kernel<<<256, 256, 0, s>>>(p->d_cb, sums, counts, w, n);
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

// Sums, counts and squared distance from a dense code array codes[r][p].  A workgroup takes one
// part, as many of its columns (the count is one more) as LDS holds sums for - 64-bit ones, see
// vq_nearest.hip - and every ny-th strip of rows, and writes its sums to the workspace:
// sums [ny][P][w][len], counts [ny][P][len]; or adds them to the one (zeroed) set there is room for.
// Before, every value was an atomic on memory (1.1 M per part and round at 65 536 rows of 16
// columns) and every wave one on the distortion: 1.7 ms of a round's 2.8 at 8 x 2048 x 16.
constexpr int kAccThreads = 1024;
constexpr int64_t kAccLds = 144 * 1024;

template <typename T, typename CODE>
__global__ __launch_bounds__(kAccThreads) void vq_accumulate_codes_kernel(
    const T *__restrict__ x, int64_t rows, int D, int w, int len, int P, const CODE *__restrict__ codes,
    const float *__restrict__ cb, int DG, int groups, int ny, int one_set, float *__restrict__ sums,
    uint32_t *__restrict__ counts, double *__restrict__ distortion) {
    extern __shared__ double s_acc[];  // [DG][len]
    __shared__ double s_dist;
    const int grp = blockIdx.x % groups, p = blockIdx.x / groups % P, by = blockIdx.x / (groups * P);
    const int c0 = grp * DG, nc = min(DG, w + 1 - c0);  // columns c0.. ; column w counts
    for (int i = threadIdx.x; i < nc * len; i += kAccThreads) s_acc[i] = 0.0;
    if (threadIdx.x == 0) s_dist = 0.0;
    __syncthreads();
    float dsum = 0.0f;
    for (int64_t r = (int64_t)by * kAccThreads + threadIdx.x; r < rows; r += (int64_t)ny * kAccThreads) {
        const int code = codes[r * P + p];
        const float *ent = cb + ((int64_t)p * len + code) * w;
#pragma unroll 4
        for (int j = 0; j < nc; j++) {
            const int d = c0 + j, col = p * w + d;
            if (d < w) {
                const float xv = col < D ? load1(x + r * D + col) : 0.0f;
                unsafeAtomicAdd(&s_acc[(int64_t)j * len + code], (double)xv);
                const float diff = xv - ent[d];
                dsum += diff * diff;
            } else {
                unsafeAtomicAdd(&s_acc[(int64_t)j * len + code], 1.0);
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) dsum += __shfl_xor(dsum, o);
    if ((threadIdx.x & 63) == 0) unsafeAtomicAdd(&s_dist, (double)dsum);
    __syncthreads();
    if (threadIdx.x == 0) unsafeAtomicAdd(distortion, s_dist);
    for (int i = threadIdx.x; i < nc * len; i += kAccThreads) {
        const int j = i / len, e = i - j * len, d = c0 + j;
        if (one_set) {
            if (s_acc[i] == 0.0) continue;
            if (d < w) unsafeAtomicAdd(&sums[((int64_t)p * w + d) * len + e], (float)s_acc[i]);
            else atomicAdd(&counts[(int64_t)p * len + e], (uint32_t)s_acc[i]);
        } else if (d < w) {
            sums[(((int64_t)by * P + p) * w + d) * len + e] = (float)s_acc[i];
        } else {
            counts[((int64_t)by * P + p) * len + e] = (uint32_t)s_acc[i];
        }
    }
}

// The generic round's workspace: the codes, then the workgroups' sums.
struct GenericPlan {
    int DG, groups, ny;
    int64_t codes_bytes, set_bytes;  // codes (rounded up), sums and counts of one workgroup row
};

GenericPlan generic_plan(const bifeat_params *p, int64_t rows) {
    const int w = p->scheme.vq_width, len = p->scheme.vq_length;
    GenericPlan g;
    g.DG = (int)(kAccLds / (8 * len));  // at least one: 16384 entries take 128 KB
    if (g.DG > w + 1) g.DG = w + 1;
    g.groups = (w + g.DG) / g.DG;
    g.DG = (w + g.groups) / g.groups;
    // about two workgroups per CU, no more than there are strips, the sums within 256 MB
    const int64_t strips = (rows + kAccThreads - 1) / kAccThreads;
    g.codes_bytes = (rows * p->P * p->cbytes + 255) / 256 * 256;
    g.set_bytes = (int64_t)4 * p->P * len * (w + 1);
    int64_t ny = 512 / ((int64_t)p->P * g.groups);
    if (ny > ((int64_t)256 << 20) / g.set_bytes) ny = ((int64_t)256 << 20) / g.set_bytes;
    if (ny > strips) ny = strips;
    g.ny = (int)(ny < 1 ? 1 : ny);
    return g;
}

// Whether a codebook that the plain fused kernel can train, and the matrix-core search does not take,
// goes through codes.  The fused kernel reads the sample once a round and is bound by its LDS float
// adds; the other way searches faster, reads twice, and the second time a workgroup has one part's
// columns of all its rows, which only a sample that the caches hold allows.  10 rounds, us, fused /
// codes: 16 384 x 1 x 64 x 64 41 700 / 2600, 65 536 x 8 x 64 x 5 4369 / 1142 (widths the fused kernel
// does not have at compile time); 65 536 x 1 x 32 x 8 522 / 354, 1000 x 96 x 32 x 8 341 / 217;
// 65 536 x 8 x 16 x 1 279 / 343, 65 536 x 8 x 16 x 4 403 / 544, 65 536 x 192 x 64 x 4 5110 / 8760.
// One and two columns are so little to read that small codebooks go through codes at any size
// (65 536 x 96 x 64 x 1 1931 / 1433; 256 entries 2393 / 2958).
bool codes_pay(const bifeat_params *p, int64_t rows) {
    const int w = p->scheme.vq_width, len = p->scheme.vq_length;
    if (w > 16 || (w & (w - 1))) return true;
    if (rows * p->P * w < (1 << 21)) return len * w >= 128 || rows <= 4096;
    return w <= 2 && len <= 64;
}

template <typename T, typename CODE>
bool accumulate_codes(bifeat_params *p, const T *x, int64_t rows, const GenericPlan &g, bool one_set, float *sums,
                      uint32_t *counts, double *dist_slot, hipStream_t s) {
    const size_t shm = sizeof(double) * (size_t)g.DG * p->scheme.vq_length;
    auto kern = vq_accumulate_codes_kernel<T, CODE>;
    if (shm > 65536 - 64 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)shm) != hipSuccess)
        return false;
    kern<<<(unsigned)(g.groups * p->P * g.ny), kAccThreads, shm, s>>>(
        x, rows, (int)p->D, p->scheme.vq_width, p->scheme.vq_length, p->P, (const CODE *)p->d_scratch, p->d_cb, g.DG,
        g.groups, g.ny, one_set, sums, counts, dist_slot);
    return true;
}

template <typename T>
hipError_t lloyd_round_generic(bifeat_params *p, const T *x, int64_t rows, double *dist_slot, hipStream_t s) {
    const int w = p->scheme.vq_width, len = p->scheme.vq_length, P = p->P;
    const int64_t books = (int64_t)P * len * w;
    const GenericPlan g = generic_plan(p, rows);
    // without room for every workgroup's sums (a stream under capture) they add to the handle's own
    // block of one set (the codes' part of the workspace is there, see below): 8 x 2048 x 16 cosine,
    // 10 rounds 2890 us so, with workspace 2980; one workgroup per part and group of columns 8690
    const bool all = (int64_t)p->scratch_bytes >= g.codes_bytes + g.ny * g.set_bytes;
    const int sets = all ? g.ny : 1;
    float *sums = all ? (float *)(p->d_scratch + g.codes_bytes) : p->d_train;
    uint32_t *counts = (uint32_t *)(sums + sets * books);
    if (!all) launch_vq_zero(p->d_train, books + (int64_t)P * len, s);
    if (p->scheme.vq_metric == BIFEAT_VQ_COSINE) launch_vq_rnorm(p, s);
    launch_vq_assign(p, x, rows, p->d_scratch, (int64_t)P * p->cbytes, s);
    const bool ok = p->cbytes == 1 ? accumulate_codes<T, uint8_t>(p, x, rows, g, !all, sums, counts, dist_slot, s)
                                   : accumulate_codes<T, uint16_t>(p, x, rows, g, !all, sums, counts, dist_slot, s);
    if (!ok) return hipGetLastError();
    launch_vq_means(p, sums, counts, sets, s);
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
    bool through_codes = !fused;
    const GenericPlan g = generic_plan(p, rows);
    if (!fused) {
        // (codes without the sums: see lloyd_round_generic)
        if (!ensure_scratch(p, (size_t)(g.codes_bytes + g.ny * g.set_bytes), s) &&
            !ensure_scratch(p, (size_t)rows * P * p->cbytes, s))
            return hipErrorOutOfMemory;
    } else if (!vq_nearest_takes(p, true) && codes_pay(p, rows)) {
        through_codes = ensure_scratch(p, (size_t)(g.codes_bytes + g.ny * g.set_bytes), s);
    }
    if (init) {
        if (dtype == BIFEAT_F32)
            vq_init_kernel<float><<<256, 256, 0, s>>>((const float *)chunk, (int)p->D, w, len, P, p->d_cb);
        else
            vq_init_kernel<__half><<<256, 256, 0, s>>>((const __half *)chunk, (int)p->D, w, len, P, p->d_cb);
    }
    vq_zero_kernel<<<1, 128, 0, s>>>(reinterpret_cast<float *>(p->d_dist), 2 * rounds);
    for (int k = 0; k < rounds; k++) {
        if (!through_codes) {
            if (dtype == BIFEAT_F32) lloyd_round(p, (const float *)chunk, rows, p->d_dist + k, s);
            else lloyd_round(p, (const __half *)chunk, rows, p->d_dist + k, s);
        } else {
            const hipError_t e = dtype == BIFEAT_F32
                                     ? lloyd_round_generic(p, (const float *)chunk, rows, p->d_dist + k, s)
                                     : lloyd_round_generic(p, (const __half *)chunk, rows, p->d_dist + k, s);
            if (e != hipSuccess) return e;
        }
    }
    return hipGetLastError();
}

}  // namespace bf
