// Streaming fit and encode+pack kernels (one-time preprocessing, paper
// Sec. 3.3; code definitions Sec. 3.1 Eq. (1) and Sec. 3.2).
//
// All three kernels stream a row-major [rows x D] chunk once.  A thread owns a
// fixed group of consecutive columns for its whole life (the grid's row stride
// is a multiple of the groups per row), so per-column parameters live in
// registers while consecutive lanes still read consecutive addresses.
#include "common.hpp"
#include "stream_kernels.hpp"
#include "vq_assign_impl.hpp"
#include "vq_nearest.hpp"

namespace bf {

// ------------------------------------------------------------------ fit state
// copy blockIdx.y of the state, `stride` words from one to the next
__global__ void fit_reset_kernel(int32_t *state, int stride, int n_half, int32_t a, int32_t b) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    state += (int64_t)blockIdx.y * stride;
    if (i < n_half) {
        state[i] = a;
        state[n_half + i] = b;
    }
}

hipError_t launch_fit_reset(bifeat_params *p, hipStream_t s) {
    if (p->scheme.kind == BIFEAT_SQ_UNIFORM) {
        int D = (int)p->D;
        fit_reset_kernel<<<dim3((D + 255) / 256, fit_copies(D)), 256, 0, s>>>(p->d_fit, 2 * D, D, kKeyPosInf, kKeyNegInf);
    } else {
        // log: [0] = smallest nonzero |x| (bits of +inf), [1] = largest finite |x| (0)
        fit_reset_kernel<<<dim3(1, kFitCopies), 64, 0, s>>>(p->d_fit, kFitMagStride, 1, 0x7F800000, 0);
    }
    return hipGetLastError();
}

// smallest nonzero and largest finite magnitude of a chunk (log scheme);
// positive floats order like their bit patterns
template <typename T, bool VEC>
__global__ __launch_bounds__(kFitThreads) void fit_log_kernel(const T *__restrict__ x, int64_t n,
                                                          int32_t *state) {
    uint32_t mmin = 0x7F800000u, mmax = 0u;
    auto take = [&](float v) {
        const uint32_t m = __float_as_uint(fabsf(v));
        if (m < 0x7F800000u) {  // finite
            if (m != 0u && m < mmin) mmin = m;
            if (m > mmax) mmax = m;
        }
    };
    if constexpr (VEC) {
        // every workgroup streams one contiguous piece of the chunk, 4 elements per lane
        const int64_t n4 = n >> 2, per_block = (n4 + gridDim.x - 1) / gridDim.x;
        const int64_t i0 = (int64_t)blockIdx.x * per_block, i1 = min(n4, i0 + per_block);
#pragma unroll 4
        for (int64_t i = i0 + threadIdx.x; i < i1; i += kFitThreads) {
            const float4 v = load4(x + 4 * i);
            take(v.x);
            take(v.y);
            take(v.z);
            take(v.w);
        }
        if (blockIdx.x == 0 && threadIdx.x < (n & 3)) take(load1(x + 4 * n4 + threadIdx.x));
    } else {
        const int64_t stride = (int64_t)gridDim.x * kFitThreads;
#pragma unroll 4
        for (int64_t i = (int64_t)blockIdx.x * kFitThreads + threadIdx.x; i < n; i += stride)
            take(load1(x + i));
    }
    merge_magnitudes(mmin, mmax, state);
}

hipError_t launch_fit_update(bifeat_params *p, const void *chunk, int dtype, int64_t rows,
                             hipStream_t s) {
    const int D = (int)p->D;
    if (p->scheme.kind == BIFEAT_SQ_LOG) {
        int64_t n = rows * D;
        const int blocks = fit_blocks((n + 31) / 32);
        const bool vec4 = (uintptr_t)chunk % (dtype == BIFEAT_F32 ? 16 : 8) == 0;
        if (dtype == BIFEAT_F32) {
            if (vec4) fit_log_kernel<float, true><<<blocks, kFitThreads, 0, s>>>((const float *)chunk, n, p->d_fit);
            else fit_log_kernel<float, false><<<blocks, kFitThreads, 0, s>>>((const float *)chunk, n, p->d_fit);
        } else {
            if (vec4) fit_log_kernel<__half, true><<<blocks, kFitThreads, 0, s>>>((const __half *)chunk, n, p->d_fit);
            else fit_log_kernel<__half, false><<<blocks, kFitThreads, 0, s>>>((const __half *)chunk, n, p->d_fit);
        }
        return hipGetLastError();
    }
    const size_t esz = dtype == BIFEAT_F32 ? 4 : 2;
    const bool vec = (D % 4 == 0) && ((uintptr_t)chunk % (4 * esz) == 0);
    if (dtype == BIFEAT_F32) return launch_fit_minmax_src(p, ChunkSrc<float>{(const float *)chunk, D}, rows, vec, s);
    return launch_fit_minmax_src(p, ChunkSrc<__half>{(const __half *)chunk, D}, rows, vec, s);
}

// scale_j = (max_j - min_j)/L and inv_j = L/(max_j - min_j): fp64 subtraction
// and division, one rounding to fp32; 0 for a constant column; zeros as +0.
__global__ void finalize_uniform_kernel(const int32_t *state, int copies, int D, int bits, float *mn,
                                        float *mx, float *scale, float *inv, float *host) {
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= D) return;
    int32_t lo_k = state[j], hi_k = state[D + j];
#pragma unroll 8
    for (int c = 1; c < copies; c++) {
        lo_k = min(lo_k, state[(int64_t)c * 2 * D + j]);
        hi_k = max(hi_k, state[(int64_t)c * 2 * D + D + j]);
    }
    float lo = key_float(lo_k), hi = key_float(hi_k);
    if (lo == 0.0f) lo = 0.0f;
    if (hi == 0.0f) hi = 0.0f;
    double L = (double)((1u << bits) - 1u);
    double range = (double)hi - (double)lo;
    mn[j] = lo;
    mx[j] = hi;
    const float s = range > 0.0 ? (float)(range / L) : 0.0f, i = range > 0.0 ? (float)(L / range) : 0.0f;
    scale[j] = s;
    inv[j] = i;
    if (host) {  // (laid out like the four above)
        host[j] = lo;
        host[D + j] = s;
        host[2 * D + j] = i;
        host[3 * D + j] = hi;
    }
}

__global__ void export_kernel(const uint32_t *__restrict__ src, uint32_t *__restrict__ dst, int words) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < words; i += gridDim.x * blockDim.x) dst[i] = src[i];
}

void launch_export(bifeat_params *p, const void *src, int words, hipStream_t s) {
    export_kernel<<<(words + 255) / 256, 256, 0, s>>>((const uint32_t *)src, (uint32_t *)p->d_out, words);
}

hipError_t launch_finalize_uniform(bifeat_params *p, hipStream_t s) {
    int D = (int)p->D;
    finalize_uniform_kernel<<<(D + 63) / 64, 64, 0, s>>>(p->d_fit, fit_copies(D), D, p->scheme.bits, p->d_min,
                                                            p->d_max, p->d_scale, p->d_inv, p->d_out);
    return hipGetLastError();
}

template <typename T>
static void launch_vq_assign(bifeat_params *p, const T *x, int64_t rows, uint8_t *codes, hipStream_t s) {
    // the matrix-core search gives the same codes
    if (!launch_vq_nearest_codes<T>(p, x, rows, codes, p->rb, p->cbytes, s)) launch_vq_plain<false>(p, x, rows, codes, s);
}

hipError_t launch_quantize(bifeat_params *p, const void *chunk, int dtype, int64_t rows,
                           uint8_t *codes, hipStream_t s) {
    const int D = (int)p->D;
    const size_t esz = dtype == BIFEAT_F32 ? 4 : 2;
    const bool vec = (D % 4 == 0) && ((uintptr_t)chunk % (4 * esz) == 0);
    if (p->scheme.kind == BIFEAT_VQ) {
        if (dtype == BIFEAT_F32) launch_vq_assign(p, (const float *)chunk, rows, codes, s);
        else launch_vq_assign(p, (const __half *)chunk, rows, codes, s);
    } else if (dtype == BIFEAT_F32) {
        return launch_quantize_sq_src(p, ChunkSrc<float>{(const float *)chunk, D}, rows, codes, vec, s);
    } else {
        return launch_quantize_sq_src(p, ChunkSrc<__half>{(const __half *)chunk, D}, rows, codes, vec, s);
    }
    return hipGetLastError();
}

}  // namespace bf
