// Nearest-entry search of the vector codes on the matrix cores: what its callers see.
#pragma once

#include "common.hpp"

namespace bf {

// Whether the matrix-core search takes the handle's shape for so many rows: not parts of more than 32 columns,
// codebooks of few values, of entries too dense for its margin or too large for LDS, nor in
// training those whose sums do not fit LDS next to the entries.  (The two
// calls below return false, with nothing launched, when it does not.)
bool vq_nearest_takes(const bifeat_params *p, bool train, int64_t rows);
// rows x parts from which on it takes some small codebooks
constexpr int64_t kNearestManyParts = 1 << 18;

// the index of every part's nearest entry: row r's part p, p->cbytes bytes, goes to codes + r * rb + p * pb.  Rows of
// a table: pb = cbytes, and the bytes from P * cbytes to rb are zeroed; one part's indices after the other (training):
// rb = cbytes, pb = rows * cbytes.
template <typename T>
bool launch_vq_nearest_codes(bifeat_params *p, const T *x, int64_t rows, uint8_t *codes, int64_t rb, int64_t pb,
                             hipStream_t s);

// one Lloyd round over the rows: every entry becomes the mean of the parts nearest to it (cosine: by
// the reciprocal norms in p->d_rnorm), their squared distances are added to *distortion
template <typename T>
bool launch_vq_nearest_round(bifeat_params *p, const T *x, int64_t rows, double *distortion, hipStream_t s);

// Training's sums.  A set's are added up in 64 bits and rounded to 32, and an entry's mean comes from the
// sets in their order: which rows make up a set decides the last bits of a codebook, and after some rounds
// which side rows between two entries fall to.  So the sets follow from the scheme and the number of rows
// alone: strip k of 2^strip_log2 rows belongs to set k % sets.  How many workgroups there are is up to the kernel:
// one takes every groups-th set, or `sub` share a set, whose sums stay in 64 bits until they have met.
struct RowSets {
    int strip_log2, sets, groups, sub;
    int64_t share;  // rows of a set that a workgroup takes, a whole number of waves
};
RowSets row_sets(const bifeat_params *p, int64_t rows);
// groups, sub and share for `cols` columns of workgroups of `threads` rows at a time, of which `room` run side by side
void deal_sets(RowSets &r, int64_t rows, int64_t cols, int64_t room, int threads);
inline int64_t sums_bytes(const bifeat_params *p, const RowSets &r) {
    return (int64_t)r.sets * r.sub * p->P * p->scheme.vq_length * ((r.sub > 1 ? 8 : 4) * p->scheme.vq_width + 4);
}
// A round's workspace: the sums and counts, then the squared distance of each of `cols` columns of r.groups
// workgroups.  They end at about the same time, and added to one double in memory they did so 20 ns one after the other:
// ten rounds on 6863 rows of 23 x 64 x 8 took 296 us instead of 238, on 6817 of 21 x 256 x 8 356 instead of 321.
inline int64_t dists_at(const bifeat_params *p, const RowSets &r) { return (sums_bytes(p, r) + 7) / 8 * 8; }
inline int64_t round_bytes(const bifeat_params *p, const RowSets &r, int64_t cols) {
    return dists_at(p, r) + 8 * cols * r.groups;
}
inline double *round_dists(const bifeat_params *p, const RowSets &r, uint8_t *sums) {
    return reinterpret_cast<double *>(sums + dists_at(p, r));
}
// how many rows a set has, and its i-th one (strips are counted in 32 bits: a 64-bit division takes 0.5 us)
__device__ inline int64_t set_rows(int set, int sets, int strip_log2, int64_t rows) {
    const uint32_t strips = (uint32_t)((rows + (1 << strip_log2) - 1) >> strip_log2), mine = (strips - set + sets - 1) / sets;
    const int64_t past = ((int64_t)(set + (mine - 1) * sets + 1) << strip_log2) - rows;
    return ((int64_t)mine << strip_log2) - (past > 0 ? past : 0);
}
__device__ inline int64_t set_row(int set, int sets, int strip_log2, int64_t i) {
    return ((set + (i >> strip_log2) * sets) << strip_log2) + (i & ((1 << strip_log2) - 1));
}

// where the last round's last kernel leaves all rounds' squared distances for the host, else nullptr.  (A kernel of its own for that
// took 3 us of each training: 1000 rows of 1 x 256 x 16 205 us, 201 so.)
inline double *last_round(const bifeat_params *p, int round) {
    return round + 1 == p->opt_vq_iters ? reinterpret_cast<double *>(p->d_out) : nullptr;
}

// every entry with members becomes their mean, from the sums [sets][sub][P][w][len] (64 bits where sub > 1, else
// 32) and counts [sets][sub][P][len]; *distortion, one of p->d_dist = the sum of the n_dists workgroups' dists (nullptr: it is there)
void launch_vq_means(bifeat_params *p, const void *sums, const uint32_t *counts, int sets, int sub, const double *dists,
                     int n_dists, double *distortion, hipStream_t s);

}  // namespace bf
