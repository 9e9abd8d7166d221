// Aggregation over fp32 rows: the layers after the first (Appendix A.1), where the
// neighbourhood mean runs over the previous layer's output instead of packed codes,
// and the row-length reduction of the scale profile (Appendix A.1, A.5).
//
// Both are row gathers bound by memory: a row of D floats is fetched whole, 16 bytes per
// lane, several rows in flight per lane.  Rows of a number of columns that is no multiple of four
// begin anywhere; their last lane then takes the row's last four columns, some of them its neighbour's too,
// with the same sums.  With 4 bytes per lane there, 147 743 rows of 101 columns took 197 us, 122 so.
#include "common.hpp"

#include <algorithm>

namespace bf {
namespace {

constexpr int kAggInFlight = 4;  // rows that a lane adds up while as many travel
constexpr int kMaxLists = 3;     // destinations of a lane group of short_lists() at most
// A list longer than kLong is not walked by one lane group (a hub's thousands of rows,
// one latency after the other, would outlast the rest of the launch): it is cut into
// pieces of kSub list entries that many groups sum side by side.  A workgroup of that
// kernel looks after kRange consecutive list entries, which at most kRange / kLong + 2
// long lists can overlap: it adds its pieces up in LDS, per list, and only then to the
// output row with atomics.  (Every piece's own atomics, 10 M of them where a third of 16 M
// list entries sits in long lists, took a tenth of the launch: 1252 us, see the end of
// long_lists().  Pieces of 256 entries instead are as fast there and half as fast at 100 000
// rows.  64-bit sums: an LDS float add takes 196 cycles per wave here, a double add 22.)
constexpr int kLong = 256;
constexpr int kRange = 2048;
constexpr int kSub = 64;
constexpr int kMaxLong = kRange / kLong + 2;
// The sums a workgroup has room for: a tile of 16-byte lanes (20 KB), which it adds up at a time.
constexpr int kSums = kMaxLong * 256;

// Compensated (Kahan) running sums: the rounding error of a sum stays at a couple of
// ulps of the mean magnitude whatever the list length; the kernel waits on memory, so
// the three extra operations per element cost nothing.  (Compiled without contraction
// or reassociation, which this relies on.)
__device__ inline void kahan_add(float &s, float &c, const float r) {
    const float y = r - c;
    const float t = s + y;
    c = (t - s) - y;
    s = t;
}

// What has been added up so far: c holds what the additions put on top of it.  Right after an
// infinite term, or one whose addition overflowed, c is not finite; the sum then is s alone.
__device__ inline double kahan_sum(const float s, const float c) {
    return __builtin_isfinite(c) ? (double)s - (double)c : (double)s;
}

template <int VEC>
struct Acc;
template <>
struct Acc<4> {
    float4 v, c;
    __device__ void zero() { v = c = make_float4(0.f, 0.f, 0.f, 0.f); }
    __device__ static float4 load(const float *p) { return load4_any(p); }
    __device__ static void hold(float4 &r) { asm volatile("" : "+v"(r.x), "+v"(r.y), "+v"(r.z), "+v"(r.w)); }
    __device__ void add(const float4 r) {
        kahan_add(v.x, c.x, r.x);
        kahan_add(v.y, c.y, r.y);
        kahan_add(v.z, c.z, r.z);
        kahan_add(v.w, c.w, r.w);
    }
    // a thread's sum of its group's k-th list, kept in LDS
    __device__ void park(double *lds, int k) const { reinterpret_cast<float4 *>(lds)[k * kThreads + threadIdx.x] = v; }
    __device__ static float4 parked(const double *lds, int k) { return reinterpret_cast<const float4 *>(lds)[k * kThreads + threadIdx.x]; }
    __device__ static void store(float4 o, float *p, int n, bool sum) {
        if (!sum) {
            const float d = (float)n;
            o = n > 0 ? make_float4(o.x / d, o.y / d, o.z / d, o.w / d) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        store4_any(p, o);
    }
    // this piece's sum, without its first `skip` columns
    __device__ void add_to(double *p, int skip) const {
        if (skip < 1) unsafeAtomicAdd(p + 0, kahan_sum(v.x, c.x));
        if (skip < 2) unsafeAtomicAdd(p + 1, kahan_sum(v.y, c.y));
        if (skip < 3) unsafeAtomicAdd(p + 2, kahan_sum(v.z, c.z));
        unsafeAtomicAdd(p + 3, kahan_sum(v.w, c.w));
    }
};
template <>
struct Acc<1> {
    float v, c;
    __device__ void zero() { v = c = 0.f; }
    __device__ static float load(const float *p) { return *p; }
    __device__ void add(const float r) { kahan_add(v, c, r); }
    __device__ static void store(float o, float *p, int n, bool sum) {
        __builtin_nontemporal_store(sum ? o : (n > 0 ? o / (float)n : 0.f), p);
    }
    __device__ void add_to(double *p, int) const { unsafeAtomicAdd(p, kahan_sum(v, c)); }
};

// a 64-bit value of the wave's lane `at / 4`
__device__ inline int64_t from_lane(int64_t v, int at) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(at, (int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(at, (int)(v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// rows of the list entries [e, end) added into acc, U loads in flight
template <int VEC, int U>
__device__ inline void add_rows(Acc<VEC> &acc, const float *__restrict__ base, int64_t D,
                                const int64_t *__restrict__ indices, int64_t e, int64_t end) {
    for (; e + U <= end; e += U) {
        decltype(Acc<VEC>::load(base)) r[U];
#pragma unroll
        for (int k = 0; k < U; k++) r[k] = Acc<VEC>::load(base + indices[e + k] * D);
#pragma unroll
        for (int k = 0; k < U; k++) acc.add(r[k]);
    }
    for (; e < end; e++) acc.add(Acc<VEC>::load(base + indices[e] * D));
}

// Of a group's lists the k-th one, with `before` entries in those ahead of it, is left to left_lists() where it would make
// the group's chain longer than one list's can be.
__device__ inline bool is_left(int k, int before, int len) { return k > 0 && len > 0 && before + len > kLong; }

// The lists of up to kLong entries.  A group of `lpr` lanes (a power of two from 8 to 64)
// owns a column tile of `lists` destinations, V / lists apart: lane t of the group accumulates
// columns 4*(tile*lpr + t) .. +3 over each destination's list, in list order
// (fp32, compensated).  Items are numbered tile-fastest.  Long lists are left to long_lists().
// What bounds it is how many rows are in flight: 2^20 rows of 100 columns, 17 M entries, ask for 6.9 GB
// beyond the L2s, which move 7.4 TB/s of such lines at most.  The group's lists are one run of entries,
// whose rows travel 4 by 4 wherever a list begins and ends (most have 3 to 8 entries),
// the next 4 while these are added.  The group fetches lpr entries with one load and hands the rows'
// places round by lane exchange; a list's sum waits in LDS until the item's rows have been
// read, as loads issued behind a store return behind it.  That launch: 1070 us with a list at a time, 4
// rows in flight and every entry loaded by all lanes, 960 so; 300 000 rows of 100 columns 271 and 234.
// Consecutive destinations instead share the loads of their bounds and entries (6 of them: 953 us a round), but lists of nearly
// kLong entries tend to be neighbours, and one group's chain of them outlasts the launch (417 408 rows of 64
// columns 318 us, 137 apart; 55 456 of 100 sorted by degree 217, 77).  Apart they meet where the numbering has a stride
// of about V / lists (rank r at (1 000 003 r + 12 345) mod V: 68 182 rows of 100 columns 126 us, 230 249 of 64 175);
// with such groups' further lists left to others 77 and 115.  Blocks of destinations paired as hashed instead: 92 there, but
// some heavy list ends every launch (200 047 rows of 64 columns 131, 115 so); left to the workgroup's
// other groups, which have as heavy ones: 126.
__device__ inline void short_lists(const float *__restrict__ x, int64_t D,
                                   const int64_t *__restrict__ indptr,
                                   const int64_t *__restrict__ indices, int64_t V, int lpr_log2,
                                   int lists, int tiles, int sum, float *__restrict__ out, int64_t block,
                                   int64_t nblocks) {
    constexpr int U = kAggInFlight;
    using Sum = Acc<4>;
    extern __shared__ double s_sum[];
    const int lpr = 1 << lpr_log2;
    const int lane = threadIdx.x & 63, t = lane & (lpr - 1), first = lane & ~(lpr - 1);
    const int64_t groups = (nblocks * kThreads) >> lpr_log2;
    const int64_t step = (V + lists - 1) / lists, items = step * tiles;
    for (int64_t item = (block * kThreads + threadIdx.x) >> lpr_log2; item < items; item += groups) {
        const int64_t v0 = item / tiles;
        const int tile = (int)(item - v0 * tiles);
        const int64_t col0 = (int64_t)4 * (tile * lpr + t), col = min(col0, D - 4);
        const bool in = col0 < D;  // (the other lanes read a row's end and write nothing)
        // lane t: the t-th destination's list (lists < lpr), none for a long one
        const int64_t v = v0 + t * step;
        const bool mine = t < lists && v < V;
        const int64_t beg = mine ? indptr[v] : 0;
        // (bounds that decrease, against the contract, leave an empty list: the others' places must not move)
        int all = mine ? (int)min(max(indptr[v + 1] - beg, (int64_t)0), (int64_t)kLong + 1) : kLong + 1;
        int len = all <= kLong ? all : 0;
        // where it begins in the run of all of them (from lane `lists` on: the run's end)
        auto begins = [&]() {
            int at = 0;
#pragma unroll
            for (int k = 0; k < kMaxLists; k++) {
                const int len_k = __builtin_amdgcn_ds_bpermute(4 * (first + k), len);
                at += t > k ? len_k : 0;
            }
            return at;
        };
        int rel = begins();
        const bool left = t < lists && is_left(t, rel, len);
        if (__any(left)) {
            if (left) { all = kLong + 1; len = 0; }
            rel = begins();
        }
        const int64_t shift = beg - rel;
        const int n = __builtin_amdgcn_ds_bpermute(4 * (first + lists), rel);
        const float *src = x + col;
        int i = 0, end = __builtin_amdgcn_ds_bpermute(4 * (first + 1), rel);
        Sum acc;
        acc.zero();
        auto close = [&]() {  // list i is complete
            acc.park(s_sum, i);
            i++;
            end = i < lists ? __builtin_amdgcn_ds_bpermute(4 * (first + i + 1), rel) : 0x7FFFFFFF;
            acc.zero();
        };
        while (end == 0) close();
        if (n > 0) {
            // place of the row of the run's e-th entry (past the last one: the last)
            auto place = [&](int e) {
                e = min(e, n - 1);
                int k = 0;
#pragma unroll
                for (int j = 1; j < kMaxLists; j++) k += e >= __builtin_amdgcn_ds_bpermute(4 * (first + j), rel);
                return indices[from_lane(shift, 4 * (first + k)) + e] * D;
            };
            // of this chunk of lpr entries, and of the next one
            int64_t off = place(t), off1 = place(lpr + t);
            float4 r[2][U];
            auto rows = [&](float4 (&to)[U], int e) {  // entries e .. e + U - 1 travel
                if (e > 0 && (e & (lpr - 1)) == 0) {
                    off = off1;
                    off1 = place(e + lpr + t);
                }
#pragma unroll
                for (int u = 0; u < U; u++)
                    to[u] = Sum::load(src + from_lane(off, 4 * (first + ((e + u) & (lpr - 1)))));
            };
            auto take = [&](float4 (&of)[U], int e) {
                // (each in registers before the first is used: the compiler would otherwise move the loads into
                // the branches, one after the other)
#pragma unroll
                for (int u = 0; u < U; u++) Sum::hold(of[u]);
                if (e + U < end) {
#pragma unroll
                    for (int u = 0; u < U; u++) acc.add(of[u]);
                } else {
#pragma unroll
                    for (int u = 0; u < U; u++) {
                        if (e + u < n) {
                            acc.add(of[u]);
                            while (e + u + 1 == end) close();
                        }
                    }
                }
            };
            rows(r[0], 0);
            for (int e = 0; e < n; e += 2 * U) {
                const bool second = e + U < n;
                if (second) rows(r[1], e + U);
                take(r[0], e);
                if (e + 2 * U < n) rows(r[0], e + 2 * U);
                if (second) take(r[1], e + U);
            }
        }
        for (int k = 0; k < lists; k++) {
            const int n_k = __builtin_amdgcn_ds_bpermute(4 * (first + k), all);  // (more than kLong: none, or a long one)
            if (in && n_k <= kLong) Sum::store(Sum::parked(s_sum, k), out + (v0 + k * step) * D + col, n_k, sum != 0);
        }
    }
}

// The lists that short_lists() leaves, a lane group each.  A lane looks one item's lists over; lanes of a wave are far apart,
// as such items tend to be neighbours.  (Another look at the bounds: 2^20 rows of 100 columns 955 us without,
// 960; 300 000 of 64 128, 131; one list after the other 133.)
__device__ inline void left_lists(const float *__restrict__ x, int64_t D, const int64_t *__restrict__ indptr,
                                  const int64_t *__restrict__ indices, int64_t V, int lpr_log2, int lists, int tiles, int sum,
                                  float *__restrict__ out, int64_t block, int64_t nblocks) {
    const int64_t step = (V + lists - 1) / lists, items = step * tiles;
    const int lane = threadIdx.x & 63, lpr = 1 << lpr_log2, t = lane & (lpr - 1);
    block = (block & 7) * (nblocks >> 3) + (block >> 3);  // (a multiple of 8: consecutive ones on one XCD)
    const int64_t wave = block * (kThreads / 64) + (threadIdx.x >> 6), waves = nblocks * (kThreads / 64);
    for (int64_t first = 0; first < items; first += 64 * waves) {
        const int64_t item = first + wave + waves * lane;
        const int64_t tile = tiles == 1 && item < items ? 0 : item / step, v0 = item - tile * step;
        int before = 0;
        bool any = false;
#pragma unroll
        for (int k = 0; k < kMaxLists; k++) {  // (all bounds at once; hardly a wave finds anything)
            const int64_t v = min(v0 + k * step, V - 1), all = indptr[v + 1] - indptr[v];
            const int len = item < items && k < lists && v0 + k * step < V && all > 0 && all <= kLong ? (int)all : 0;
            any |= is_left(k, before, len);
            before += len;
        }
        if (!__any(any)) continue;
        before = 0;
        for (int k = 0; k < lists; k++) {
            const int64_t v = v0 + k * step;
            const bool mine = item < items && v < V;
            const int64_t beg = mine ? indptr[v] : 0, all = mine ? indptr[v + 1] - beg : 0;
            const int len = all > 0 && all <= kLong ? (int)all : 0;
            const uint64_t left = __ballot(is_left(k, before, len));
            before += len;
            const int n = __popcll(left);
            for (int it0 = 0; it0 < n; it0 += 64 >> lpr_log2) {
                const int it = it0 + (lane >> lpr_log2);
                uint64_t m = left;
                for (int i = 0; i < it; i++) m &= m - 1;
                const int at = 4 * (m ? __ffsll((unsigned long long)m) - 1 : 0);
                const int64_t of = from_lane(v, at), b = from_lane(beg, at);
                const int len_of = __builtin_amdgcn_ds_bpermute(at, len);
                const int64_t col0 = 4 * (__builtin_amdgcn_ds_bpermute(at, (int)tile) * lpr + t), col = min(col0, D - 4);
                const bool in = it < n && col0 < D;
                Acc<4> acc;
                acc.zero();
                if (in) add_rows<4, 2 * kAggInFlight>(acc, x + col, D, indices, b, b + len_of);
                if (in) Acc<4>::store(acc.v, out + of * D + col, len_of, sum != 0);
            }
        }
    }
}

// The lists of up to kLong entries again, a destination at a time.  For launches that do not fill the chip several times over:
// a group each of as many lists as there are hides more than runs of them do (25 323 rows of 64 columns 42 us by
// runs, 32 so; 8500 of 32 37, 25).  And for rows that four lanes take (up to 16 columns): with 16 groups a wave some list
// ends at every row, and short_lists() then walks its slow branch (10^6 rows of 16 226, 217).  One list a group: four, far
// apart, were 3 to 15 % slower (500 000 rows of 16 columns 118 us, 105 so; 3000 of 64 33, 25).
template <int VEC>
__device__ inline void short_lists_single(const float *__restrict__ x, int64_t D,
                                          const int64_t *__restrict__ indptr,
                                          const int64_t *__restrict__ indices, int64_t V, int lpr_log2, int tiles, int sum,
                                          float *__restrict__ out, int64_t block, int64_t nblocks) {
    const int lpr = 1 << lpr_log2, t = threadIdx.x & (lpr - 1);
    const int64_t items = V * tiles, groups = (nblocks * kThreads) >> lpr_log2;
    for (int64_t item = (block * kThreads + threadIdx.x) >> lpr_log2; item < items; item += groups) {
        const int64_t v = item / tiles;
        const int tile = (int)(item - v * tiles);
        const int64_t col0 = (int64_t)VEC * (tile * lpr + t), col = min(col0, D - VEC);
        const int64_t beg = indptr[v], end = indptr[v + 1];
        if (col0 >= D || end - beg > kLong) continue;
        Acc<VEC> acc;
        acc.zero();
        add_rows<VEC, kAggInFlight>(acc, x + col, D, indices, beg, end);
        Acc<VEC>::store(acc.v, out + v * D + col, (int)(end - beg), sum != 0);
    }
}

// The long lists: a workgroup looks after kRange consecutive list entries at a time.  It
// finds the first destination whose list reaches into that range (a 64-way search in
// indptr by one wave), walks on from there, notes the long lists with the part that
// falls inside the range, and its lane groups sum pieces of kSub entries of those parts.
// The lists' sums over the range go to the output rows, which aggregate_zero_long_kernel
// has zeroed.
template <int VEC>
__device__ inline void long_lists(const float *__restrict__ x, int64_t D,
                                  const int64_t *__restrict__ indptr,
                                  const int64_t *__restrict__ indices, int64_t V, int64_t E,
                                  int lpr_log2, int tiles, int sum, float *__restrict__ out,
                                  int64_t block, int64_t nblocks) {
    __shared__ int64_t s_v[kMaxLong], s_beg[kMaxLong], s_end[kMaxLong], s_first;
    __shared__ int s_deg[kMaxLong], s_n;
    extern __shared__ double s_sum[];  // [long lists][columns of a tile]
    const int lpr = 1 << lpr_log2;
    const int t = threadIdx.x & (lpr - 1);
    const int group = threadIdx.x >> lpr_log2, groups = kThreads >> lpr_log2;
    constexpr int kPieces = kRange / kSub;
    for (int64_t r0 = block * kRange; r0 < E; r0 += nblocks * kRange) {
        const int64_t r1 = r0 + kRange < E ? r0 + kRange : E;
        if (threadIdx.x < 64) {
            // first v with indptr[v + 1] > r0: 64 probes a round, evenly spaced over [lo, hi)
            int64_t lo = 0, hi = V;
            while (lo < hi) {
                const int64_t step = (hi - lo + 63) >> 6;
                const int64_t probe = lo + (int64_t)threadIdx.x * step;
                const uint64_t valid = __ballot(probe < hi);
                const uint64_t hit = __ballot(probe < hi && indptr[probe + 1] > r0);
                if (hit == 0) {
                    lo += (int64_t)(__popcll(valid) - 1) * step + 1;  // past the last probe
                } else {
                    const int j = __ffsll((unsigned long long)hit) - 1;
                    hi = lo + j * step;
                    if (j > 0) lo += (int64_t)(j - 1) * step + 1;
                }
            }
            if (threadIdx.x == 0) {
                s_first = lo;
                s_n = 0;
            }
        }
        __syncthreads();
        // walk the destinations from there until one starts at or after r1
        for (int64_t v0 = s_first;; v0 += kThreads) {
            const int64_t v = v0 + threadIdx.x;
            bool past = v >= V;
            if (!past) {
                const int64_t beg = indptr[v];
                past = beg >= r1;
                if (!past) {
                    const int64_t end = indptr[v + 1];
                    if (end - beg > kLong) {
                        const int k = atomicAdd(&s_n, 1);
                        if (k < kMaxLong) {
                            s_v[k] = v;
                            s_beg[k] = beg > r0 ? beg : r0;
                            s_end[k] = end < r1 ? end : r1;
                            s_deg[k] = (int)(end - beg);
                        }
                    }
                }
            }
            if (__syncthreads_or(past)) break;
        }
        const int n_long = s_n < kMaxLong ? s_n : kMaxLong;
        const int tile_cols = lpr * VEC;
        for (int tile = 0; tile < tiles && n_long > 0; tile++) {
            for (int i = threadIdx.x; i < n_long * tile_cols; i += kThreads) s_sum[i] = 0.0;
            __syncthreads();
            for (int it = group; it < n_long * kPieces; it += groups) {
                const int piece = it % kPieces, k = it / kPieces;
                const int64_t b = s_beg[k] + (int64_t)piece * kSub;
                const int64_t col0 = (int64_t)VEC * (tile * lpr + t), col = min(col0, D - VEC);
                if (b >= s_end[k]) continue;
                const bool in = col0 < D;
                Acc<VEC> acc;
                acc.zero();
                if (in) add_rows<VEC, 2 * kAggInFlight>(acc, x + col, D, indices, b, min(b + kSub, s_end[k]));
                const int skip = (int)(col0 - col);
                if (in) acc.add_to(s_sum + k * tile_cols + VEC * t - skip, skip);
            }
            __syncthreads();
            for (int i = threadIdx.x; i < n_long * tile_cols; i += kThreads) {
                const int k = i / tile_cols;
                const int64_t col = (int64_t)tile * tile_cols + (i - k * tile_cols);
                if (col < D)
                    unsafeAtomicAdd(out + s_v[k] * D + col, (float)(sum ? s_sum[i] : s_sum[i] / (double)s_deg[k]));
            }
            __syncthreads();
        }
        __syncthreads();
    }
}

// One launch for all: the first `long_blocks` workgroups (dispatched first; their
// pieces are the longest single chains of the launch) take the long lists, the rest
// the short ones, one or, where `lists` is not 0, several at a time, those that these leave first.  All write disjoint rows.
template <int VEC, bool SINGLE>
__device__ inline void aggregate(const float *__restrict__ x, int64_t D, const int64_t *__restrict__ indptr,
                                 const int64_t *__restrict__ indices, int64_t V, int64_t E, int lpr_log2, int lists,
                                 int left_blocks, int tiles, int sum, int long_blocks, float *__restrict__ out) {
    const int64_t block = (int64_t)blockIdx.x - long_blocks, nblocks = (int64_t)gridDim.x - long_blocks;
    if (block < 0)
        long_lists<VEC>(x, D, indptr, indices, V, E, lpr_log2, tiles, sum, out, blockIdx.x, long_blocks);
    else if constexpr (SINGLE)
        short_lists_single<VEC>(x, D, indptr, indices, V, lpr_log2, tiles, sum, out, block, nblocks);
    else if (block < left_blocks)
        left_lists(x, D, indptr, indices, V, lpr_log2, lists, tiles, sum, out, block, left_blocks);
    else
        short_lists(x, D, indptr, indices, V, lpr_log2, lists, tiles, sum, out, block - left_blocks, nblocks - left_blocks);
}
#define BF_AGG(NAME, VEC, SINGLE)                                                                            \
    void NAME(const float *__restrict__ x, int64_t D, const int64_t *__restrict__ indptr,                     \
              const int64_t *__restrict__ indices, int64_t V, int64_t E, int lpr_log2, int lists, int left_blocks, \
              int tiles, int sum, int long_blocks, float *__restrict__ out) {                                 \
        aggregate<VEC, SINGLE>(x, D, indptr, indices, V, E, lpr_log2, lists, left_blocks, tiles, sum, long_blocks, out); \
    }
// (apart: with the registers of short_lists() a SIMD holds 5 waves instead of 8, and the narrow
// lists, 10^6 rows of 8 columns, take 210 us instead of 197)
__global__ __launch_bounds__(kThreads) BF_AGG(aggregate_rows_kernel, 4, false)
__global__ __launch_bounds__(kThreads) BF_AGG(aggregate_rows_single_kernel4, 4, true)
__global__ __launch_bounds__(kThreads) BF_AGG(aggregate_rows_single_kernel1, 1, true)
#undef BF_AGG

// Output rows of the long lists set to zero ahead of the launch above: a lane per
// destination looks at its list length, the wave then clears each long one's row.
__global__ __launch_bounds__(kThreads) void aggregate_zero_long_kernel(
    const int64_t *__restrict__ indptr, int64_t V, int64_t D, float *__restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    // whole waves stay in the loop together: the bound is rounded up to the wave
    for (int64_t v0 = (int64_t)blockIdx.x * kThreads + (threadIdx.x & ~63); v0 < V; v0 += stride) {
        const int64_t v = v0 + lane;
        const bool is_long = v < V && indptr[v + 1] - indptr[v] > kLong;
        uint64_t m = __ballot(is_long);
        while (m) {
            const int j = __ffsll((unsigned long long)m) - 1;
            m &= m - 1;
            float *row = out + (v0 + j) * D;
            for (int64_t c = lane; c < D; c += 64) row[c] = 0.f;
        }
    }
}

// acc[0] += sum over rows of sqrt(sum_j h[i][j]^2): one wave per row, squares and
// their sum in fp64, one atomic per workgroup.
template <int VEC>
__global__ __launch_bounds__(kThreads) void row_length_sum_kernel(const float *__restrict__ h,
                                                                  int64_t n, int64_t D,
                                                                  double *__restrict__ acc) {
    __shared__ double s_part[kThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t waves = (int64_t)gridDim.x * (kThreads / 64);
    double total = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * (kThreads / 64) + wave; i < n; i += waves) {
        const float *row = h + i * D;
        double q = 0.0;
        if constexpr (VEC == 4) {
            for (int64_t j = 4 * lane; j < D; j += 256) {
                const float4 r = *reinterpret_cast<const float4 *>(row + j);
                q += (double)r.x * r.x;
                q += (double)r.y * r.y;
                q += (double)r.z * r.z;
                q += (double)r.w * r.w;
            }
        } else {
            for (int64_t j = lane; j < D; j += 64) q += (double)row[j] * row[j];
        }
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) q += __shfl_xor(q, m, 64);
        total += sqrt(q);
    }
    if (lane == 0) s_part[wave] = total;
    __syncthreads();
    if (threadIdx.x == 0) {
        double b = 0.0;
        for (int k = 0; k < kThreads / 64; k++) b += s_part[k];
        if (b != 0.0) atomicAdd(acc, b);
    }
}

bool vec_ok(const void *a, const void *b, int64_t D) {
    return D % 4 == 0 && (uintptr_t)a % 16 == 0 && (uintptr_t)b % 16 == 0;
}

}  // namespace

hipError_t launch_aggregate_rows(const float *x, int64_t D, const int64_t *indptr,
                                 const int64_t *indices, int64_t V, int64_t E, int sum, float *out,
                                 hipStream_t s) {
    // 16 bytes a lane.  Rows of few columns that begin anywhere: 4 bytes where there are not many, more lanes
    // then share a hub's (us by 16 bytes / 4: 20 000 rows of 30 columns 48 / 31, of 15 32 / 29; 200 000 of 15 71 / 65, of 23
    // 92 / 92, 500 000 of 15 136 / 153, of 30 181 / 246; 20 000 of 33 44 / 46)
    const bool vec = D >= 4 && (D % 4 == 0 || D > 32 || V >= (D > 16 ? 1 << 17 : 1 << 18));
    const int64_t granules = vec ? (D + 3) / 4 : D;
    int lpr_log2 = 2;  // at least four lanes per row
    while (lpr_log2 < 6 && ((int64_t)1 << lpr_log2) < granules) lpr_log2++;
    const int64_t tiles = (granules + ((int64_t)1 << lpr_log2) - 1) >> lpr_log2;
    // Several lists a group only where the chip has enough of them at a time (us with 1, 2, 3 of them: 2^20
    // rows of 64 columns 776, 680, 595, of 100 1174, 1017, 973; 417 408 of 100 354, 336, 334; 114 390 of 64, 29 000
    // waves by one, 85, 74, 72).  Rows of 64 lanes: 100 000 of 256 columns 154, 160, 167, 196 516 304, 271, 273; 100 000 of 768
    // 512, 548, 570, 500 000 of 300 two 1322, three 1239.  0: short_lists_single().  Fewer than 4 entries a list on
    // average end too often for two (none / 2: 50 021 rows of 64 columns, 2.3 entries, 28 / 40, 50 000 of 100, 2 each, 15.5 / 17.0, 114 390 of 64,
    // 3.6, 54 / 59; but by three 200 047 of 64, 3.6, 72 / 66), fewer than 2 for three up to 256 MB of sums (400 000 of 100, one each, 69 / 79;
    // but 2^20 of 100, 1.5 each, 298 / 248).
    const int64_t waves = (V * tiles) >> (6 - lpr_log2);
    int lists = !vec || lpr_log2 == 2 || waves < (E < 4 * V ? 32768 : 12288) ||
                        (E < 2 * V && V * D <= (int64_t)1 << 26)         ? 0
                : waves < 32768 || (lpr_log2 == 6 && V < (int64_t)1 << 17) ? 2
                                                                         : kMaxLists;
    // (no more than make one list of kLong on average: what is left is dearer; 100 000 rows of 100 columns and 120 entries
    // each 766 us by two, 1180 by three)
    if (lists * E > kLong * V) lists = 2 * E > kLong * V ? 0 : 2;
    const int64_t step = lists ? (V + lists - 1) / lists : V, items = step * tiles;
    // many small workgroups rather than one resident set: the two kinds of work take turns
    // on the CUs as slots free up, and no workgroup's share is large enough to form a tail
    const int short_blocks = blocks_for(items << lpr_log2, 1 << 20);
    const int left_blocks = lists ? (blocks_for(items, 1 << 20) + 7) / 8 * 8 : 0;
    int long_blocks = 0;
    if (E > kLong) {  // otherwise no list is long
        const int64_t ranges = (E + kRange - 1) / kRange;
        long_blocks = (int)(ranges < (1 << 20) ? ranges : (1 << 20));
        aggregate_zero_long_kernel<<<blocks_for(V, 8 * 256), kThreads, 0, s>>>(indptr, V, D, out);
    }
    const int blocks = short_blocks + left_blocks + long_blocks;
    const int64_t tile_cols = (int64_t)(vec ? 4 : 1) << lpr_log2;
    size_t shm = long_blocks > 0 ? sizeof(double) * (size_t)std::min<int64_t>(kSums, kMaxLong * tile_cols) : 0;
    shm = std::max(shm, (size_t)lists * kThreads * 16);  // the short lists' sums
    auto *kern = lists ? aggregate_rows_kernel : vec ? aggregate_rows_single_kernel4 : aggregate_rows_single_kernel1;
    kern<<<blocks, kThreads, shm, s>>>(x, D, indptr, indices, V, E, lpr_log2, lists, left_blocks, (int)tiles, sum, long_blocks, out);
    return hipGetLastError();
}

// a small fill kernel instead of a memset node: callers may capture the stream into a graph
__global__ void zero_doubles_kernel(double *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0;
}

void launch_zero_doubles(double *p, int n, hipStream_t s) {
    zero_doubles_kernel<<<(n + 127) / 128, 128, 0, s>>>(p, n);
}

hipError_t launch_row_length_sum(const float *h, int64_t n, int64_t D, double *acc, hipStream_t s) {
    const int blocks = blocks_for(n * 64, 8 * 256);
    if (vec_ok(h, h, D))
        row_length_sum_kernel<4><<<blocks, kThreads, 0, s>>>(h, n, D, acc);
    else
        row_length_sum_kernel<1><<<blocks, kThreads, 0, s>>>(h, n, D, acc);
    return hipGetLastError();
}

}  // namespace bf
