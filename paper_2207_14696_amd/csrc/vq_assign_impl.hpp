// Plain nearest-entry search of the vector codes, for what the matrix-core search leaves (wide parts, tiny
// codebooks, dense ones and those that do not fit LDS).  Its two layouts of the codes have a file each: a
// file's kernels are loaded together, at the first launch of one, and most processes that encode never train.
#pragma once

#include "common.hpp"

namespace bf {

namespace {

// Vector codes (Sec. 3.2): workgroup = one part x strips of 256 rows, thread =
// one row whose sub-vector stays in registers; the part's codebook passes
// through LDS in chunks of EC entries (all of it at once when it fits), read
// by all threads at the same address (broadcast).  Euclidean: fp32, dims
// ascending, subtract / multiply / add rounded separately, strict < keeps the
// lowest index on ties.  Cosine: fp32 dot product accumulated the same way,
// times the entry's reciprocal norm, strict > keeps the lowest index.
// W > 0: the width, known at compile time; W == 0: any width up to WMAX.
// PARTS: codes part after part, not rows of rb bytes (the two strides as arguments are two more scalar
// registers to spill: 65 536 rows of 8 x 1200 x 30 cosine 3290 us, 2890 so).
template <typename T, int W, int WMAX, int METRIC, typename CODE, bool PARTS>
__global__ __launch_bounds__(kThreads) void vq_assign_kernel(
    const T *__restrict__ x, int64_t rows, int D, int w_rt, int len, int P, int EC,
    const float *__restrict__ cb, const float *__restrict__ rnorm, uint8_t *__restrict__ codes,
    int64_t rb) {
    extern __shared__ float s_cb[];
    const int w = W > 0 ? W : w_rt;
    float *s_rn = s_cb + EC * w;
    const int p = blockIdx.x;
    const float *part_cb = cb + (int64_t)p * len * w;
    const bool single = len <= EC;
    auto stage = [&](int e0, int ec) {
        for (int i = threadIdx.x; i < ec * w; i += kThreads) s_cb[i] = part_cb[(int64_t)e0 * w + i];
        if constexpr (METRIC == BIFEAT_VQ_COSINE)
            for (int i = threadIdx.x; i < ec; i += kThreads) s_rn[i] = rnorm[(int64_t)p * len + e0 + i];
    };
    if (single) {
        stage(0, len);
        __syncthreads();
    }
    // every thread of the workgroup walks the same strips (the chunk loads synchronise)
    for (int64_t r0 = (int64_t)blockIdx.y * kThreads; r0 < rows; r0 += (int64_t)gridDim.y * kThreads) {
        const int64_t r = r0 + threadIdx.x;
        const bool valid = r < rows;
        float sub[WMAX];
        if (W % 4 == 0 && W > 0 && p * W + W <= D) {  // (a row of 64 lanes is 64 lines, whatever is loaded of each)
#pragma unroll
            for (int d = 0; d < WMAX; d += 4) {
                const float4 q = valid ? load4_any(x + r * D + (int64_t)p * W + d) : make_float4(0.f, 0.f, 0.f, 0.f);
                sub[d] = q.x; sub[(d + 1) % WMAX] = q.y; sub[(d + 2) % WMAX] = q.z; sub[(d + 3) % WMAX] = q.w;
            }
        } else {
#pragma unroll
            for (int d = 0; d < WMAX; d++)
                sub[d] = (valid && d < w && p * w + d < D) ? load1(x + r * D + (int64_t)p * w + d) : 0.0f;
        }
        int best = 0;
        float bestv = METRIC == BIFEAT_VQ_COSINE ? -INFINITY : INFINITY;
        for (int e0 = 0; e0 < len; e0 += EC) {
            const int ec = min(EC, len - e0);
            if (!single) {
                __syncthreads();
                stage(e0, ec);
                __syncthreads();
            }
            for (int c = 0; c < ec; c++) {
                const float *ent = s_cb + c * w;
                float acc = 0.0f;
#pragma unroll
                for (int d = 0; d < WMAX; d++) {
                    if (W > 0 || d < w) {  // uniform; sub[] stays in registers
                        if constexpr (METRIC == BIFEAT_VQ_COSINE) {
                            acc = __fadd_rn(acc, __fmul_rn(sub[d], ent[d]));
                        } else {
                            const float diff = __fsub_rn(sub[d], ent[d]);
                            acc = __fadd_rn(acc, __fmul_rn(diff, diff));
                        }
                    }
                }
                if constexpr (METRIC == BIFEAT_VQ_COSINE) {
                    acc = __fmul_rn(acc, s_rn[c]);
                    if (acc > bestv) { bestv = acc; best = e0 + c; }
                } else {
                    if (acc < bestv) { bestv = acc; best = e0 + c; }
                }
            }
        }
        if (valid) {
            if constexpr (PARTS) {
                reinterpret_cast<CODE *>(codes)[p * rows + r] = (CODE)best;
            } else {
                reinterpret_cast<CODE *>(codes + r * rb)[p] = (CODE)best;
                if (p == 0)
                    for (int64_t b = (int64_t)P * sizeof(CODE); b < rb; b++) codes[r * rb + b] = 0;  // row padding
            }
        }
    }
}

template <bool PARTS, typename T, int W, int WMAX>
void launch_vq_w(bifeat_params *p, const T *x, int64_t rows, uint8_t *codes, hipStream_t s) {
    const int w = p->scheme.vq_width, len = p->scheme.vq_length;
    const bool cosine = p->scheme.vq_metric == BIFEAT_VQ_COSINE;
    int EC = 32768 / (4 * w);  // entries per LDS chunk: 32 KB of entries
    if (EC > len) EC = len;
    int64_t tiles = (rows + kThreads - 1) / kThreads;
    dim3 grid((unsigned)p->P, (unsigned)(tiles > 4096 ? 4096 : tiles));
    const size_t shm = sizeof(float) * ((size_t)EC * w + (cosine ? EC : 0));
#define BF_VQ(M, CODE)                                                                   \
    vq_assign_kernel<T, W, WMAX, M, CODE, PARTS><<<grid, kThreads, shm, s>>>(           \
        x, rows, (int)p->D, w, len, p->P, EC, p->d_cb, p->d_rnorm, codes, p->rb)
    if (p->cbytes == 1) {
        if (cosine) BF_VQ(BIFEAT_VQ_COSINE, uint8_t);
        else BF_VQ(BIFEAT_VQ_L2, uint8_t);
    } else {
        if (cosine) BF_VQ(BIFEAT_VQ_COSINE, uint16_t);
        else BF_VQ(BIFEAT_VQ_L2, uint16_t);
    }
#undef BF_VQ
}

template <bool PARTS, typename T>
void launch_vq_plain(bifeat_params *p, const T *x, int64_t rows, uint8_t *codes, hipStream_t s) {
    const int w = p->scheme.vq_width;
    switch (w) {
        case 1: launch_vq_w<PARTS, T, 1, 1>(p, x, rows, codes, s); break;
        case 2: launch_vq_w<PARTS, T, 2, 2>(p, x, rows, codes, s); break;
        case 4: launch_vq_w<PARTS, T, 4, 4>(p, x, rows, codes, s); break;
        case 8: launch_vq_w<PARTS, T, 8, 8>(p, x, rows, codes, s); break;
        case 16: launch_vq_w<PARTS, T, 16, 16>(p, x, rows, codes, s); break;
        default:
            if (w <= 32) launch_vq_w<PARTS, T, 0, 32>(p, x, rows, codes, s);
            else if (w <= 64) launch_vq_w<PARTS, T, 0, 64>(p, x, rows, codes, s);
            else launch_vq_w<PARTS, T, 0, 128>(p, x, rows, codes, s);
            break;
    }
}

}  // namespace

}  // namespace bf
