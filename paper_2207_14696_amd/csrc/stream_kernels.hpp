// The streaming kernels of the one-time preprocessing (paper Sec. 3.3; code definitions
// Sec. 3.1 Eq. (1)), written against a *row source* instead of a pointer: the per-column
// range fit, the fit of the extreme magnitudes, and encode + pack of the scalar codes.
//
// A row source hands out the table's values; it is either a chunk resident in memory
// (ChunkSrc, what bifeat_fit_update / bifeat_quantize take) or a producer that makes the
// values on the fly (anything with the same three members, instantiated by the caller's
// own translation unit through include/bifeat_produce.hpp) - then the raw table never
// exists in memory at all, neither for the fit nor for the encoder (Appendix D: the
// preprocessing cost is one pass to fit and one to encode).
//
//   struct Src {
//       struct Ctx;                                        // per-thread state of a column group
//       __device__ void prepare(Ctx &, int col0, int D) const;   // once per thread
//       __device__ float4 load4(const Ctx &, int64_t r, int col0) const;  // columns col0..col0+3 of row r
//       __device__ float load1(const Ctx &, int64_t r, int col) const;    // one column of row r
//   };
// (the chunk source has load4_any as well, and load8 for half-precision chunks)
//
// In all kernels a thread owns a fixed group of consecutive columns for its whole life (the
// grid's row stride is a multiple of the groups per row), so per-column parameters live in
// registers while consecutive lanes still touch consecutive addresses.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace bf {

// rows of a chunk in memory, row-major, element type T (float or __half)
template <typename T>
struct ChunkSrc {
    const T *x;
    int D;
    struct Ctx {};
    __device__ void prepare(Ctx &, int, int) const {}
    __device__ float4 load4(const Ctx &, int64_t r, int col0) const { return bf::load4(x + r * D + col0); }
    __device__ float4 load4_any(const Ctx &, int64_t r, int col0) const { return bf::load4_any(x + r * D + col0); }
    __device__ float load1(const Ctx &, int64_t r, int col) const { return bf::load1(x + r * D + col); }
    __device__ void load8(const Ctx &, int64_t r, int col0, float (&v)[8]) const { bf::load8(x + r * D + col0, v); }
};

template <class Src>
constexpr bool kChunk = false;
template <typename T>
constexpr bool kChunk<ChunkSrc<T>> = true;
template <class Src>
constexpr bool kHalfChunk = std::is_same<Src, ChunkSrc<__half>>::value;

// The fit kernels end with atomics on a few words (2*D of them, or two, in kFitCopies copies), and the
// workgroups of a launch come to that end together: 2048 workgroups of 256 threads spent 80 of 210 us there
// (a 524 288 x 768 half-precision chunk and one copy; the read alone takes 130).  So there are few workgroups,
// of 1024 threads: two per CU.  That chunk's range with its reset: 245 -> 168 us; the extreme
// magnitudes of 1 M x 128 floats 234 -> 102 us, of half-precision values 210 -> 51 us (4 atomics a
// workgroup on two words before, at most 2 now).
constexpr int kFitThreads = 1024;
constexpr int kFitBlocks = 512;

// A workgroup's rows of a chunk come in pieces of so many of its iterations, the workgroups' pieces one after the
// other: the chip then reads one window of the chunk at a time (2^20 x 1024 half precision 360 us with one long piece each,
// 336 so).  The last round's rows are dealt evenly (90 000 x 768 half precision: by pieces of this length too a tenth of the
// workgroups could have them all, 32 us, 27 so).  Whole pieces have a number of iterations that the compiler knows: worked out for
// each, with a 64-bit division, pieces of 16 cost more than they gave (2^20 x 128 floats 88 us with one long piece, 93, and 84 so).
// Not a power of two, which the iterations' 16 KB often are (2^20 x 256 floats by 16 of them 176, by 20 167; by 12, 28 or 40 as by 20).
// Half precision by 16 bytes whose iterations are no whole number of 4 KB: 8 loads at a time (524 288 x 768 135 us by 4, 133 so, 2^20 x 896
// 304 and 298; but 2^20 x 512 170 and 178, floats by 8 a tenth slower).
constexpr int kFitPiece = 20, kFitPieceBy8 = 32;

inline int fit_blocks(int64_t threads) {
    const int64_t b = (threads + kFitThreads - 1) / kFitThreads;
    return (int)(b < 1 ? 1 : b > kFitBlocks ? kFitBlocks : b);
}

// smallest nonzero and largest finite magnitude seen by a workgroup merged into state[0], [1]: one
// atomic each, and none that would change nothing (positive floats order like their bits)
__device__ inline void merge_magnitudes(uint32_t mmin, uint32_t mmax, int32_t *state) {
    __shared__ uint32_t s_mm[2];
    if (threadIdx.x == 0) {
        s_mm[0] = 0x7F800000u;
        s_mm[1] = 0u;
    }
    __syncthreads();
    for (int o = 32; o > 0; o >>= 1) {
        mmin = min(mmin, (uint32_t)__shfl_xor((int)mmin, o));
        mmax = max(mmax, (uint32_t)__shfl_xor((int)mmax, o));
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMin(&s_mm[0], mmin);
        atomicMax(&s_mm[1], mmax);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t *st = reinterpret_cast<uint32_t *>(state) + blockIdx.x % kFitCopies * kFitMagStride;
        if (s_mm[0] < __builtin_nontemporal_load(&st[0])) atomicMin(&st[0], s_mm[0]);
        if (s_mm[1] > __builtin_nontemporal_load(&st[1])) atomicMax(&st[1], s_mm[1]);
    }
}

// per-column min / max of the rows [0, rows) of `src` merged into the running state.
// VEC = 4 needs D % 4 == 0 (and, for a chunk in memory, 16-byte / 8-byte alignment), VEC = 8 (half
// precision in memory) D % 8 == 0 and 16 bytes.  TH: threads of a workgroup, see the launcher.
template <class Src, int VEC, int TH>
__global__ __launch_bounds__(TH) void fit_minmax_kernel(Src src, int64_t rows, int D, int G, int32_t *state,
                                                        int use_lds) {
    extern __shared__ int32_t lds[];
    if (use_lds) state += blockIdx.x % kFitCopies * 2 * D;
    if (use_lds) {
        for (int i = threadIdx.x; i < D; i += TH) {
            lds[i] = kKeyPosInf;
            lds[D + i] = kKeyNegInf;
        }
        __syncthreads();
    }
    // A workgroup takes TH/G whole rows per iteration when a row's G column groups fit it (a wave's
    // lanes then read consecutive 16 bytes), else groups of G threads across the grid walk consecutive rows - also
    // where single columns would leave more than a quarter of the workgroup idle (601 half-precision
    // columns, 700 000 rows: 176 us so, 223 with one row per workgroup of 1024), and wider groups two
    // fifths (204 400 rows of 2052 floats 278 us, 300; but 4 194 of 3000 12.1, 10.1).
    const bool by_block = G <= TH && TH % G <= (VEC > 1 ? 2 * TH / 5 : TH / 4);
    const int rpi = by_block ? TH / G : 0;  // rows per iteration of a workgroup
    const uint32_t total = gridDim.x * TH;
    const uint32_t rows_per_pass = total / (uint32_t)G;
    const uint32_t t = blockIdx.x * TH + threadIdx.x;
    const bool active = by_block ? (int)threadIdx.x < rpi * G : t < rows_per_pass * (uint32_t)G;
    if (active) {
        const int g = by_block ? (int)threadIdx.x % G : (int)(t % (uint32_t)G);
        float mn[VEC], mx[VEC];
#pragma unroll
        for (int k = 0; k < VEC; k++) {
            mn[k] = INFINITY;
            mx[k] = -INFINITY;
        }
        typename Src::Ctx ctx;
        src.prepare(ctx, g * VEC, D);
        // fminf / fmaxf pass over a NaN like the comparisons they stand for
        auto take = [&](int64_t r) {
            float v[VEC];
            if constexpr (VEC == 8) {
                src.load8(ctx, r, g * VEC, v);
            } else if constexpr (VEC == 4) {
                float4 q = src.load4(ctx, r, g * VEC);
                v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
            } else {
                v[0] = src.load1(ctx, r, g);
            }
#pragma unroll
            for (int k = 0; k < VEC; k++) {
                mn[k] = fminf(mn[k], v[k]);
                mx[k] = fmaxf(mx[k], v[k]);
            }
        };
        if (by_block) {
            const int row = (int)threadIdx.x / G;
            const bool by8 = VEC == 8 && rpi * D * 2 % 4096 != 0;
            const int steps = by8 ? kFitPieceBy8 : kFitPiece;
            const int64_t round = (int64_t)gridDim.x * rpi * steps;
            int64_t base = 0;
            if constexpr (kChunk<Src>) {
                for (; base + round <= rows; base += round) {
                    const int64_t r0 = base + (int64_t)blockIdx.x * (rpi * steps) + row;
                    if (by8) {
#pragma unroll 8
                        for (int k = 0; k < kFitPieceBy8; k++) take(r0 + k * rpi);
                    } else {
#pragma unroll 4
                        for (int k = 0; k < kFitPiece; k++) take(r0 + k * rpi);
                    }
                }
            }
            const int64_t pass = (int64_t)gridDim.x * rpi, piece = (rows - base + pass - 1) / pass * rpi;
            const int64_t r0 = base + blockIdx.x * piece, end = min(rows, r0 + piece);
#pragma unroll 4
            for (int64_t r = r0 + row; r < end; r += rpi) take(r);
        } else {
            const int64_t K = (rows + rows_per_pass - 1) / rows_per_pass;
            const int64_t rbeg = (int64_t)(t / G) * K, rend = min(rows, rbeg + K);
#pragma unroll 4
            for (int64_t r = rbeg; r < rend; r++) take(r);
        }
        // one or two column groups: the lanes of a wave that share one merge first (the same few
        // words of LDS for all of a workgroup's atomics: 3 M rows of 4 half-precision columns 17 us, 9 so)
        bool merged = false;
        if (by_block && G <= 2) {
            for (int m = 32; m >= G; m >>= 1) {
#pragma unroll
                for (int k = 0; k < VEC; k++) {
                    mn[k] = fminf(mn[k], __shfl_xor(mn[k], m));
                    mx[k] = fmaxf(mx[k], __shfl_xor(mx[k], m));
                }
            }
            merged = (int)(threadIdx.x & 63) >= G;
        }
        // (two loops: through one pointer to either the atomics would be flat ones)
        if (!merged && use_lds) {
#pragma unroll
            for (int k = 0; k < VEC; k++) {
                atomicMin(&lds[g * VEC + k], float_key(mn[k]));
                atomicMax(&lds[D + g * VEC + k], float_key(mx[k]));
            }
        } else if (!merged) {
#pragma unroll
            for (int k = 0; k < VEC; k++) {
                atomicMin(&state[g * VEC + k], float_key(mn[k]));
                atomicMax(&state[D + g * VEC + k], float_key(mx[k]));
            }
        }
    }
    if (use_lds) {
        __syncthreads();
        // thousands of workgroups would hammer the same 2*D words: only those that improve
        // on the value already there (read without ordering: a stale read merely costs one
        // atomic that changes nothing) issue the atomic
        for (int i = threadIdx.x; i < D; i += TH) {
            const int32_t lo_k = lds[i], hi_k = lds[D + i];
            if (lo_k < __builtin_nontemporal_load(&state[i])) atomicMin(&state[i], lo_k);
            if (hi_k > __builtin_nontemporal_load(&state[D + i])) atomicMax(&state[D + i], hi_k);
        }
    }
}

// smallest nonzero and largest finite magnitude of the rows [0, rows) of a row source (log
// scheme); positive floats order like their bit patterns.  Thread = one group of VEC columns,
// rows interleaved across the grid.
template <class Src, int VEC>
__global__ __launch_bounds__(kFitThreads) void fit_log_rows_kernel(Src src, int64_t rows, int D, int G,
                                                               int32_t *state) {
    uint32_t mmin = 0x7F800000u, mmax = 0u;
    auto take = [&](float v) {
        const uint32_t m = __float_as_uint(fabsf(v));
        if (m < 0x7F800000u) {  // finite
            if (m != 0u && m < mmin) mmin = m;
            if (m > mmax) mmax = m;
        }
    };
    const uint32_t total = gridDim.x * kFitThreads;
    const uint32_t rows_per_pass = total / (uint32_t)G;
    const uint32_t t = blockIdx.x * kFitThreads + threadIdx.x;
    if (t < rows_per_pass * (uint32_t)G) {
        const int g = (int)(t % (uint32_t)G);
        typename Src::Ctx ctx;
        src.prepare(ctx, g * VEC, D);
#pragma unroll 4
        for (int64_t r = t / G; r < rows; r += rows_per_pass) {
            if constexpr (VEC == 4) {
                const float4 v = src.load4(ctx, r, g * VEC);
                take(v.x);
                take(v.y);
                take(v.z);
                take(v.w);
            } else {
                take(src.load1(ctx, r, g));
            }
        }
    }
    merge_magnitudes(mmin, mmax, state);
}

// ------------------------------------------------------------ scalar encoders
struct UniformCoder {
    static constexpr bool kEdges = false;
    const float *mn, *inv;
    float L;
    template <int NC> struct Ctx { float mn[NC], inv[NC]; };
    // VEC: D % 4 == 0
    template <bool VEC, int NC>
    __device__ void prepare(Ctx<NC> &c, int col0, int D) const {
        // 16 bytes a load where that goes: by 4 bytes the lanes' loads, NC columns apart, cross so many
        // lines that 8 columns' parameters took 8 us at the head of a launch (25 MB of half-precision
        // values 6.9 us, 18.5 before; 4 columns a lane that way: 10)
        if constexpr (VEC) {
#pragma unroll
            for (int k = 0; k < NC; k += 4) {
                const int j = min(col0 + k, D - 4);  // (past D: not used)
                const float4 m = *reinterpret_cast<const float4 *>(mn + j);
                const float4 s = *reinterpret_cast<const float4 *>(inv + j);
                c.mn[k] = m.x; c.mn[k + 1] = m.y; c.mn[k + 2] = m.z; c.mn[k + 3] = m.w;
                c.inv[k] = s.x; c.inv[k + 1] = s.y; c.inv[k + 2] = s.z; c.inv[k + 3] = s.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < NC; k++) {
                const int j = min(col0 + k, D - 1);
                c.mn[k] = mn[j];
                c.inv[k] = inv[j];
            }
        }
    }
    // q = clamp(rne((x - min) * inv), 0, L); sub, mul, round are separate fp32
    // operations; max/min discard NaN, so NaN -> 0
    template <int BITS, int NC>
    __device__ uint32_t code(const Ctx<NC> &c, float x, int k) const {
        float d = __fsub_rn(x, c.mn[k]);
        float t = __fmul_rn(d, c.inv[k]);
        float r = rintf(t);
        r = fminf(fmaxf(r, 0.0f), L);
        return (uint32_t)(int)r;
    }
};

struct LogCoder {
    static constexpr bool kEdges = true;
    const float *T;  // global, H-1 edges
    int H;
    // level l lies near a*log2|x| + b; a = 0: the range is too narrow or too extreme for that
    float a, b;
    template <int NC> struct Ctx { const float *edges; };
    template <bool VEC, int NC>
    __device__ void prepare(Ctx<NC> &c, int, int) const { c.edges = nullptr; }
    // l = #{i : |x| >= T_i}: the level the hardware's logarithm gives, put right against the edges
    // on both sides of it.  With a <= 1024 and magnitudes whose logarithm is no denormal's, the
    // logarithm (an ulp, 2^-17 at most) and b (2^-6) are off by far less than a level, the
    // fp32 edges by 2^-23, so one step either way is enough.  Otherwise by bisection.
    // edges (in LDS): [-1, T_1 .. T_{H-1}, NaN]; a NaN takes level 0 both ways.
    // 524 288 x 768 half-precision values to 4 bits: 257 us, bisection 374; 262 144 x 768 to 8 bits:
    // 129 us, bisection 361.
    // (a single edge, 2 bits, is a comparison: 105 us for 1 M x 128 floats, by the logarithm 110)
    template <int BITS, int NC>
    __device__ uint32_t code(const Ctx<NC> &c, float x, int) const {
        constexpr int H = 1 << (BITS - 1);
        float m = fabsf(x);
        int lo = 0;
        if constexpr (BITS <= 2) {
            if (BITS == 2 && m >= c.edges[1]) lo = 1;
        } else if (a > 0.0f) {
            const int l = (int)fmaf(__builtin_amdgcn_logf(m), a, b);
            lo = min(max(l, 0), H - 1);
            const float below = c.edges[lo], above = c.edges[lo + 1];
            lo += (m >= above ? 1 : 0) - (m < below ? 1 : 0);
        } else {
            int hi = H - 1;
            while (lo < hi) {
                int mid = (lo + hi) >> 1;
                if (m >= c.edges[mid + 1]) lo = mid + 1; else hi = mid;
            }
        }
        return (uint32_t)((x > 0.0f) ? H + lo : H - 1 - lo);
    }
};

// One thread encodes NC consecutive columns (NC*BITS bits): 4, or 8 of a half-precision chunk (one
// 16-byte load).  Where that is less than a 32-bit word, neighbouring lanes OR their pieces
// together and one of them stores it.  Every word of the padded row is written (columns >= D
// encode as 0).  Bound by memory (a plain copy moves 4.9 TB/s here): 524 288 x 768 half-precision
// values to 4 bits 186 us, 5.4 TB/s (8-byte loads: 221), to 1 bit 177 (206).
// stream: streaming stores, see launch_sq.
template <class Src, int BITS, typename Coder, bool VEC, int NC>
__global__ __launch_bounds__(kThreads) void quantize_sq_kernel(Src src, int64_t rows, int D, int64_t rb,
                                                              Coder coder, int stream,
                                                              uint8_t *__restrict__ codes) {
    __shared__ float s_edges[130];
    typename Coder::template Ctx<NC> ctx;
    constexpr int LG = NC * BITS >= 32 ? 1 : 32 / (NC * BITS);  // lanes per 32-bit word
    constexpr int NW = NC * BITS > 32 ? NC * BITS / 32 : 1;     // words per lane
    constexpr int CPW = NC / NW;                                // columns of a lane per word
    // Columns of a row from which on rows that begin anywhere are loaded by fours, below which the lanes without columns of
    // a padded row wait for as much work (us by single columns / so: 1 M x 21 floats to 1 bit 49 / 55, to 1 logarithmic one 41 / 54,
    // 1 M x 5 to 4 15.7 / 17.3, but 1 M x 9 to 2 bits 41 / 30; half precision to 1 bit 1 M x 5 71 / 56).
    [[maybe_unused]] constexpr int kFours = kHalfChunk<Src> ? 4 : BITS == 1 || (Coder::kEdges && BITS >= 4) ? 40 : 7;
    const int GW = (int)(8 * rb / (NC * BITS));  // NC-column groups per padded row; a multiple of LG
    if constexpr (Coder::kEdges) {
        for (int i = threadIdx.x; i <= coder.H; i += kThreads)
            s_edges[i] = i == 0 ? -1.0f : i < coder.H ? coder.T[i - 1] : __builtin_nanf("");
        __syncthreads();
    }
    const uint32_t total = gridDim.x * kThreads;
    const uint32_t rows_per_pass = total / (uint32_t)GW;
    const uint32_t t = blockIdx.x * kThreads + threadIdx.x;
    if (t >= rows_per_pass * (uint32_t)GW) return;
    const int g = (int)(t % (uint32_t)GW);
    const int col0 = NC * g;
    coder.template prepare<VEC>(ctx, col0, D);
    if constexpr (Coder::kEdges) ctx.edges = s_edges;
    typename Src::Ctx sctx;
    src.prepare(sctx, col0, D);
    const int sub = g % LG;
    uint32_t *dst_word = reinterpret_cast<uint32_t *>(codes) + (int64_t)(g / LG) * NW;
    const int64_t rw = rb / 4;
    // rows interleaved across the grid: a wave's stores stay contiguous (consecutive rows
    // per thread, as in the fit kernel, measured 15 % slower here; four rows of a thread loaded
    // ahead of their stores: 10-25 % slower)
    for (int64_t r = t / GW; r < rows; r += rows_per_pass) {
        float v[NC];
#pragma unroll
        for (int k = 0; k < NC; k++) v[k] = 0.0f;
        if constexpr (VEC && NC == 8) {
            if (col0 < D) src.load8(sctx, r, col0, v);
        } else if constexpr (VEC) {
            if (col0 < D) {
                float4 q = src.load4(sctx, r, col0);
                v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
            }
        } else if (kChunk<Src> && D >= kFours) {
            // rows that begin anywhere; the last lane takes the row's last four columns (200 000 x 602
            // floats to 4 logarithmic bits 148 us by single columns, 119 so; 66 901 x 602 half precision to 1 bit 34, 25)
            if constexpr (kChunk<Src>) {
                if (col0 < D) {
                    const float4 q = src.load4_any(sctx, r, min(col0, D - 4));
                    const int skip = col0 + 4 - D;  // of them; what is past D is not used
                    v[0] = skip <= 0 ? q.x : skip == 1 ? q.y : skip == 2 ? q.z : q.w;
                    v[1] = skip <= 0 ? q.y : skip == 1 ? q.z : q.w;
                    v[2] = skip <= 0 ? q.z : q.w;
                    v[3] = q.w;
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < NC; k++)
                if (col0 + k < D) v[k] = src.load1(sctx, r, col0 + k);
        }
        uint32_t word[NW];
#pragma unroll
        for (int n = 0; n < NW; n++) {
            word[n] = 0u;
#pragma unroll
            for (int k = 0; k < CPW; k++) {
                const int j = n * CPW + k;
                const uint32_t q = (VEC ? col0 < D : col0 + j < D) ? coder.template code<BITS>(ctx, v[j], j) : 0u;
                word[n] |= q << (BITS * k);
            }
        }
        if constexpr (LG > 1) {
            word[0] <<= (NC * BITS) * sub;
#pragma unroll
            for (int o = 1; o < LG; o <<= 1) word[0] |= (uint32_t)__shfl_xor((int)word[0], o);
        }
        if (sub == 0) {
            if (NC * BITS >= 16 && stream) {  // (whole lines of a wave's codes)
                // (a place that is another one to the compiler, which would make one ordinary store of this one and the one below)
                int64_t at = r * rw;
                asm volatile("" : "+v"(at));
                uint32_t *dst = dst_word + at;
                if constexpr (NW == 2) store_stream(reinterpret_cast<uint2 *>(dst), make_uint2(word[0], word[1]));
                else store_stream(dst, word[0]);
                asm volatile("");
            } else {
                uint32_t *dst = dst_word + r * rw;
                if constexpr (NW == 2) *reinterpret_cast<uint2 *>(dst) = make_uint2(word[0], word[1]);
                else *dst = word[0];
            }
        }
    }
}

template <class Src, typename Coder>
inline void launch_sq(const Src &src, int64_t rows, int D, int64_t rb, int bits, Coder coder,
                      uint8_t *codes, bool vec, hipStream_t s) {
    bool vec8 = false;
    // (8-bit uniform codes, whose stores then take 8 bytes a lane: 1.6 GB 476 us by 4 columns, 505 by 8)
    if constexpr (kHalfChunk<Src>)
        vec8 = vec && D % 8 == 0 && (uintptr_t)src.x % 16 == 0 && (bits < 8 || Coder::kEdges);
    const int GW = (int)(8 * rb / ((vec8 ? 8 : 4) * bits));
    int64_t want = (rows * GW + 1) / 2;
    if (want < GW) want = GW;
    int blocks = blocks_for(want);
    if ((int64_t)blocks * kThreads < GW) blocks = (GW + kThreads - 1) / kThreads;
    // Codes that fill much of the 256 MB cache are streamed past it: written back from there they slow down what comes
    // next, unless that is the first gather from them, which then finds them there.  Ordinary stores / streamed, us, for
    // 768 columns of half precision to 4 bits: the next range fit, of as many rows, and a first gather of 65 536 and of
    // 300 000 rows: 32 MB of codes 33 / 31, 38 / 54, 147 / 191; 48 MB 50 / 43, 38 / 54, 153 / 213; 64 MB 68 / 55, 46 / 53, 185 / 232;
    // 80 MB 82 / 64, 49 / 53, 214 / 234; 100 MB 96 / 77, 52 / 54, 225 / 237; 128 MB 112 / 95, 53 / 53, 235 / 239.
    const bool stream = rows * rb > ((int64_t)80 << 20);
    // The kernel does so where a wave's codes make whole lines (streamed by 32 or 64 bytes, 2^20 x 768 floats to 1 bit took 680 us,
    // 648 not so, half precision 349 and 340).
#define BF_QK(B, VECV, NC) \
    quantize_sq_kernel<Src, B, Coder, VECV, NC><<<blocks, kThreads, 0, s>>>(src, rows, D, rb, coder, stream, codes)
#define BF_Q(B)                                                                                 \
    do {                                                                                        \
        if constexpr (kHalfChunk<Src>) {                                                        \
            if (vec8) {                                                                         \
                BF_QK(B, true, 8);                                                              \
                break;                                                                          \
            }                                                                                   \
        }                                                                                       \
        if (vec) BF_QK(B, true, 4);                                                             \
        else BF_QK(B, false, 4);                                                                \
    } while (0)
    switch (bits) {
        case 1: BF_Q(1); break;
        case 2: BF_Q(2); break;
        case 4: BF_Q(4); break;
        default: BF_Q(8); break;
    }
#undef BF_Q
#undef BF_QK
}

// ---- launchers over a row source (scalar kinds)
// the per-column range fit (uniform codes); vec: groups of 4 columns per thread
template <class Src>
inline hipError_t launch_fit_minmax_src(bifeat_params *p, const Src &src, int64_t rows, bool vec,
                                        hipStream_t s) {
    const int D = (int)p->D;
    const int use_lds = D <= kFitCopiesColumns;
    // (columns merged without LDS, an atomic per thread and column: twice as many of them by 8 columns,
    // 5 242 rows of 20 000 half-precision columns 63 us, 185 by 8; few columns, merged in few words of
    // LDS: 524 288 rows of 24 6.4 us, 8.9 by 8)
    bool vec8 = false;
    if constexpr (kHalfChunk<Src>)
        vec8 = use_lds && D >= 64 && vec && D % 8 == 0 && (uintptr_t)src.x % 16 == 0;
    const int VEC = vec8 ? 8 : vec ? 4 : 1;
    const int G = (D + VEC - 1) / VEC;
    int64_t want = (rows * G + 7) / 8;  // about 8 rows per thread
    if (want < G) want = G;
    // few large workgroups for the sake of their merge (see above), but not where there is none, nor,
    // with few columns to merge, for chunks that would not occupy the CUs (half precision, large / small
    // ones: 300 x 768 6.5 / 4.9 us, 40 000 x 128 5.8 / 4.6, 15 000 x 768 6.8 / 7.5; but 300 x 4096
    // floats 4.9 / 7.3)
    const bool large = use_lds && (want > kThreads * 640 || G > kThreads);
    const int threads = large ? kFitThreads : kThreads;
    int blocks = large ? fit_blocks(want) : blocks_for(want);
    if ((int64_t)blocks * threads < G) blocks = (G + threads - 1) / threads;
    const size_t shm = use_lds ? sizeof(int32_t) * 2 * (size_t)D : 0;
#define BF_FM(V)                                                                                               \
    do {                                                                                                       \
        if (large) fit_minmax_kernel<Src, V, kFitThreads><<<blocks, threads, shm, s>>>(src, rows, D, G, p->d_fit, use_lds); \
        else fit_minmax_kernel<Src, V, kThreads><<<blocks, threads, shm, s>>>(src, rows, D, G, p->d_fit, use_lds); \
    } while (0)
    if constexpr (kHalfChunk<Src>) {
        if (vec8) {
            BF_FM(8);
            return hipGetLastError();
        }
    }
    if (vec) BF_FM(4);
    else BF_FM(1);
#undef BF_FM
    return hipGetLastError();
}

// the fit of the extreme magnitudes (logarithmic codes without clipping)
template <class Src>
inline hipError_t launch_fit_log_src(bifeat_params *p, const Src &src, int64_t rows, bool vec,
                                     hipStream_t s) {
    const int D = (int)p->D;
    const int VEC = vec ? 4 : 1;
    const int G = (D + VEC - 1) / VEC;
    int64_t want = (rows * G + 7) / 8;
    if (want < G) want = G;
    int blocks = fit_blocks(want);
    if ((int64_t)blocks * kFitThreads < G) blocks = (G + kFitThreads - 1) / kFitThreads;
    if (vec) fit_log_rows_kernel<Src, 4><<<blocks, kFitThreads, 0, s>>>(src, rows, D, G, p->d_fit);
    else fit_log_rows_kernel<Src, 1><<<blocks, kFitThreads, 0, s>>>(src, rows, D, G, p->d_fit);
    return hipGetLastError();
}

// encode + pack `rows` rows of a row source into the packed rows starting at codes_row0
template <class Src>
inline hipError_t launch_quantize_sq_src(bifeat_params *p, const Src &src, int64_t rows,
                                         uint8_t *codes_row0, bool vec, hipStream_t s) {
    const int D = (int)p->D;
    if (p->scheme.kind == BIFEAT_SQ_UNIFORM) {
        UniformCoder c{p->d_min, p->d_inv, (float)((1u << p->scheme.bits) - 1u)};
        launch_sq(src, rows, D, p->rb, p->scheme.bits, c, codes_row0, vec, s);
    } else {
        const int H = 1 << (p->scheme.bits - 1);
        const double a = H / (p->e_max - p->e_min);  // levels per factor of two
        const bool near = a <= 1024.0 && p->e_min >= -120.0 && p->e_max <= 127.0;  // (not NaN, not inf)
        LogCoder c{p->d_T, H, near ? (float)a : 0.0f, near ? (float)(-a * p->e_min) : 0.0f};
        launch_sq(src, rows, D, p->rb, p->scheme.bits, c, codes_row0, vec, s);
    }
    return hipGetLastError();
}

}  // namespace bf
