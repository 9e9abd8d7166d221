// Fused gather + neighbourhood mean for uniform scalar codes, short lists: which of its kernels runs.  Those for
// output rows that are 8-byte aligned only have a file of their own, because a file's kernels are loaded
// together, at the first launch of one: a process's first mean of rows that need none of them took 29 ms with
// them in this file, 20 so.
#include "gather_mean_lean_impl.hpp"

namespace bf {

static int cap64(int cap) { return cap < 64 ? cap : 64; }

// longest list the short-list kernel takes, in its narrow and wide forms
int lean_capacity(int bits, bool wide) {
    switch (bits) {
        case 8: return cap64(LeanSwar<8, false>::kCap);
        case 4: return cap64(wide ? LeanSwar<4, true>::kCap : LeanSwar<4, false>::kCap);
        case 2: return cap64(LeanSwar<2, false>::kCap);
        default: return cap64(wide ? LeanSwar<1, true>::kCap : LeanSwar<1, false>::kCap);
    }
}

// Launches the short-list kernel (lists of more than `lo` and at most `thr` rows; wide =
// the form with the larger field capacity); returns false (nothing launched) when the
// table's shape is outside what it handles.  vec: the output rows are 16-byte aligned, else 8-byte.
bool launch_gather_mean_lean(bifeat_params *p, const MeanCall &c, int thr, bool wide, int lo,
                             bool alone, bool vec) {
    return vec ? launch_lean<false>(p, c, thr, wide, lo, alone) : launch_gather_mean_lean_odd(p, c, thr, wide, lo, alone);
}

// 2-bit logarithmic codes (Sec. 3.1 Eq. (1)/(2) with k = 2): code q = 2*b1 + b0 decodes to
// -v1, -v0, +v0, +v1, so the decoded sum over a list of n rows is
//   v0*(S1 - S0) + v1*(S1 + S0 - n),   S0 = sum of b0, S1 = sum of b1,
// i.e. (v1 - v0)*S0 - n*v1  +  (v0 + v1)*S1: linear in the two bit-plane sums.  The packed row
// is therefore read as 2*D one-bit columns (bit 2t = b0, bit 2t+1 = b1 of column t) by the
// 1-bit kernel, with those two affine maps as per-bit-column parameters (p->d_min / d_scale,
// 2*D entries each), and the epilogue adds each pair.
bool launch_gather_mean_lean_log2(bifeat_params *p, const MeanCall &c, int thr, bool wide, int lo,
                                  bool alone) {
    return wide ? launch_lean_bits<1, true, true, false>(p, c, thr, lo, alone, p->d_min, p->d_scale)
                : launch_lean_bits<1, false, true, false>(p, c, thr, lo, alone, p->d_min, p->d_scale);
}

}  // namespace bf
