// Nearest-entry search over half-precision rows.
#include "vq_nearest_impl.hpp"

namespace bf {

BF_VN(__half)

}  // namespace bf
