// Nearest-entry search over float rows, which shapes it takes, and the means of a training round.  The rows'
// types are files of their own because a file's kernels are loaded together, at the first launch of one:
// a process's first training of 96 x 256 x 8 on 65 536 rows took 7.6 to 8.6 ms with both in one
// file, 5.4 to 6.6 so.
#include "vq_nearest_impl.hpp"

namespace bf {

namespace {

// An entry becomes the mean of its members (one without members keeps its value) from the
// workgroups' sums; GROUPS threads per column of an entry, each adding every GROUPS-th set in the sets'
// order.  One thread to all of the sets that few parts give (64 of 6 x 64 x 4) waits for one load after
// the other: 20 us of a round's 35.
template <int GROUPS>
__global__ __launch_bounds__(kThreads) void vq_means_kernel(const void *__restrict__ sums,
                                                            const uint32_t *__restrict__ counts, int sets, int sub, int P,
                                                            int w, int len, const double *__restrict__ dists, int n_dists,
                                                            double *__restrict__ distortion, int round, double *host,
                                                            float *__restrict__ cb) {
    constexpr int OUT = kThreads / GROUPS;
    const int first = dists || host ? 1 : 0, workers = (int)gridDim.x - first;
    if ((int)blockIdx.x < first) {  // one more workgroup, beside those of the means
        __shared__ double s_d[kThreads / 64];
        if (host && (int)threadIdx.x < round + (dists ? 0 : 1)) host[threadIdx.x] = distortion[threadIdx.x];
        if (!dists) return;
        double d = 0.0;
#pragma unroll 4
        for (int i = threadIdx.x; i < n_dists; i += kThreads) d += dists[i];
        for (int o = 32; o > 0; o >>= 1) d += __shfl_xor(d, o);
        if ((threadIdx.x & 63) == 0) s_d[threadIdx.x >> 6] = d;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int k = 1; k < kThreads / 64; k++) d += s_d[k];
            distortion[round] = d;
            if (host) host[round] = d;
        }
        return;
    }
    __shared__ double s_sum[GROUPS > 1 ? kThreads : 1];
    __shared__ uint64_t s_count[GROUPS > 1 ? kThreads : 1];
    const int64_t n = (int64_t)P * w * len;
    const int o = threadIdx.x % OUT, g = threadIdx.x / OUT;
    for (int64_t i0 = (int64_t)((int)blockIdx.x - first) * OUT; i0 < n; i0 += (int64_t)workers * OUT) {
        const int64_t i = i0 + o;
        const int e = (int)(i % len);
        const int64_t pd = i / len, p = pd / w;
        const int d = (int)(pd - p * w);
        double sum = 0.0;
        uint64_t count = 0;
        if (i < n && sub == 1) {
#pragma unroll 4
            for (int k = g; k < sets; k += GROUPS) {
                sum += (double)static_cast<const float *>(sums)[k * n + i];
                count += counts[((int64_t)k * P + p) * len + e];
            }
        } else if (i < n) {
            for (int k = g; k < sets; k += GROUPS) {
                double set = 0.0;
#pragma unroll 4
                for (int64_t j = (int64_t)k * sub; j < (int64_t)(k + 1) * sub; j++) {
                    set += static_cast<const double *>(sums)[j * n + i];
                    count += counts[(j * P + p) * len + e];
                }
                sum += (double)(float)set;
            }
        }
        if constexpr (GROUPS > 1) {
            s_sum[threadIdx.x] = sum;
            s_count[threadIdx.x] = count;
            __syncthreads();
            if (g == 0) {
#pragma unroll
                for (int k = 1; k < GROUPS; k++) {
                    sum += s_sum[k * OUT + o];
                    count += s_count[k * OUT + o];
                }
            }
            __syncthreads();
        }
        if (g == 0 && i < n && count > 0) cb[(p * len + e) * w + d] = (float)(sum / (double)count);
    }
}

}  // namespace

// Entries that lie too densely for the margin leave most rows open, and those are searched by the
// rule one entry after the other.  The distance to the nearest of `len` entries in w dimensions is
// about len^(-2/w) of M, and the gap to the next about 2/w of that: with the margin above a
// hundredth of it (4096 entries of 4 columns: 1857 us against 1499; any one-column codebook of
// some size) the plain search is the better one.  So it is for codebooks whose pieces do not fit LDS
// at once (16384 x 16: 2.7 ms against 4.9), for those of under 64 values, of under 512 in parts of
// under 4 columns (65 536 x 24 parts of 2 columns, 64 entries: 29 us against 38), and for those of under
// 384 (512 in fewer than 48 entries) where rows x parts are so few that staging is most of the call
// and the plain search has the width at compile time (4096 x 24 parts of 4 columns, 32 entries: 6.8 us
// against 8.0; 65 536 x 24: 37 against 24; 4096 x 24 parts of 12 columns, 32 entries: 27.6 against 11.9;
// 4096 x 6 parts of 16 columns, 31 entries: 9.7 against 10.6; of 8 columns, 60 entries: 10.8 against 9.6).
bool vq_nearest_takes(const bifeat_params *p, bool train, int64_t rows) {
    const int w = p->scheme.vq_width, len = p->scheme.vq_length;
    const int G = (w + 7) / 8, tiles = (len + 31) / 32;
    const bool few = rows * p->P < kNearestManyParts && (w == 4 || w == 8 || w == 16);
    if (w > kNearestMaxWidth || w * len < (w < 4 ? kNearestMinBook : few ? kNearestMinBookFew : kNearestMinBookAny))
        return false;
    if (few && len < 48 && w * len < kNearestMinBook) return false;
    if (nearest_lds(p, G, tiles, false, false) > kCuLds - 4096) return false;
    if (too_dense(w, len, w)) return false;
    return !train || entries_in_lds(p, true);
}

void launch_vq_means(bifeat_params *p, const void *sums, const uint32_t *counts, int sets, int sub, const double *dists,
                     int n_dists, double *distortion, hipStream_t s) {
    const int w = p->scheme.vq_width, len = p->scheme.vq_length;
    const int64_t n = (int64_t)p->P * len * w;
    const int round = (int)(distortion - p->d_dist);
    double *const host = last_round(p, round);
#define BF_VM(GROUPS) \
    vq_means_kernel<GROUPS><<<blocks_for(GROUPS * n) + (dists || host ? 1 : 0), kThreads, 0, s>>>( \
        sums, counts, sets, sub, p->P, w, len, dists, n_dists, p->d_dist, round, host, p->d_cb)
    // (a thread each where that fills the chip: 10 sets of 96 x 256 x 8 take 6.5 us so, 13 by groups)
    if (sets * sub > 8 && n < (1 << 16)) BF_VM(8);
    else BF_VM(1);
#undef BF_VM
}

BF_VN(float)

}  // namespace bf
