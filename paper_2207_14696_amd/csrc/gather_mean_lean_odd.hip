// The short-list mean for output rows that are 8-byte aligned only.
#include "gather_mean_lean_impl.hpp"

namespace bf {

bool launch_gather_mean_lean_odd(bifeat_params *p, const MeanCall &c, int thr, bool wide, int lo, bool alone) {
    return launch_lean<true>(p, c, thr, wide, lo, alone);
}

}  // namespace bf
