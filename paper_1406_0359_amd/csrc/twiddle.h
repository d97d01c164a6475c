// Inter-pass twiddles of the line transforms, W[m] = exp(-2 pi i m / n), from a staged table.
#pragma once

#include "common.h"

namespace purify {

// FP32 lines of 4096 and more take their inter-pass twiddles from two short tables,
// W[m] = W[(m >> LB) 2^LB] W[m mod 2^LB] (2^LB + n / 2^LB entries instead of n; a twiddle then
// carries the roundings of two entries and of their product, RMS 4.1e-8 against 2.1e-8), so a
// workgroup's LDS is little more than its line buffers and two workgroups fit on a CU.  At 2048
// the full table fits beside the lines, so its accuracy is kept there (the short tables: 2048^2,
// 10^6 visibilities, Phi^dagger Phi 378 -> 366 us).
template <typename T, int LOGN>
constexpr bool twiddles_split() { return sizeof(T) == 4 && LOGN >= 12; }
template <typename T, int LOGN>
constexpr int split_lb() { return (LOGN + 1) / 2; }
// entries of the staged table, and the full table's entry that sits at place i of it
template <typename T, int LOGN>
constexpr int twiddle_entries() {
    if constexpr (twiddles_split<T, LOGN>()) return (1 << split_lb<T, LOGN>()) + (1 << (LOGN - split_lb<T, LOGN>()));
    else return 1 << LOGN;
}
template <typename T, int LOGN>
__device__ __forceinline__ int twiddle_entry(int i) {
    if constexpr (twiddles_split<T, LOGN>()) {
        constexpr int LB = split_lb<T, LOGN>(), L = 1 << LB;
        return i < L ? i : (i - L) << LB;
    } else {
        return i;
    }
}
// apply(r, W[r k STEP]), 0 < r < R: the twiddles of one butterfly.  Of split tables each is the
// product of its own two entries; steps that are multiples of the low table's length need the
// high table alone (its product would be with 1).  Forming four of a radix-8 butterfly's seven as
// products of the other three halves the LDS reads (4096^2 column passes 452 -> 431 us adjoint,
// 428 -> 419 forward) but doubles their error (RMS 4.1e-8 -> 9.0e-8), so it is not done.
template <typename T, int LOGN, int R, int STEP, typename Fn>
__device__ __forceinline__ void twiddles(const cpx<T>* W, int k, Fn apply) {
#pragma unroll
    for (int r = 1; r < R; ++r) {
        const int m = r * k * STEP;
        if constexpr (twiddles_split<T, LOGN>()) {
            constexpr int LB = split_lb<T, LOGN>(), L = 1 << LB;
            if constexpr (STEP % L == 0) apply(r, W[L + (m >> LB)]);
            else apply(r, W[L + (m >> LB)] * W[m & (L - 1)]);
        } else {
            apply(r, W[m]);
        }
    }
}

}  // namespace purify
