// Nearest-entry search of the vector codes on the matrix cores: what its callers see.
#pragma once

#include "common.hpp"

namespace bf {

// Whether the matrix-core search takes the handle's shape for so many rows: not parts of more than 32 columns,
// codebooks of few values, of entries too dense for its margin or too large for LDS, nor in
// training those whose sums do not fit LDS next to the entries.  (The two
// calls below return false, with nothing launched, when it does not.)
bool vq_nearest_takes(const bifeat_params *p, bool train, int64_t rows);

// the index of every part's nearest entry, see launch_vq_assign
template <typename T>
bool launch_vq_nearest_codes(bifeat_params *p, const T *x, int64_t rows, uint8_t *codes, int64_t rb, int64_t pb,
                             hipStream_t s);

// one Lloyd round over the rows: every entry becomes the mean of the parts nearest to it (cosine: by
// the reciprocal norms in p->d_rnorm), their squared distances are added to *distortion
template <typename T>
bool launch_vq_nearest_round(bifeat_params *p, const T *x, int64_t rows, double *distortion, hipStream_t s);

// every entry with members becomes their mean, from ny sets of sums [P][w][len] and counts [P][len]
void launch_vq_means(bifeat_params *p, const float *sums, const uint32_t *counts, int ny, hipStream_t s);

}  // namespace bf
