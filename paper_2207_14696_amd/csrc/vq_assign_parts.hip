// Nearest entries of a training round through codes: one part's after the other.
#include "vq_assign_impl.hpp"
#include "vq_nearest.hpp"

namespace bf {

template <typename T>
void launch_vq_assign_parts(bifeat_params *p, const T *x, int64_t rows, uint8_t *codes, hipStream_t s) {
    if (!launch_vq_nearest_codes<T>(p, x, rows, codes, p->cbytes, rows * p->cbytes, s)) launch_vq_plain<true>(p, x, rows, codes, s);
}
template void launch_vq_assign_parts<float>(bifeat_params *, const float *, int64_t, uint8_t *, hipStream_t);
template void launch_vq_assign_parts<__half>(bifeat_params *, const __half *, int64_t, uint8_t *, hipStream_t);

}  // namespace bf
