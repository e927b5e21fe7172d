// One part of the kernel instances of the axis-by-axis FFT solve, so that the
// parts compile side by side: DNSLAB_PART_T the real type, DNSLAB_PART_X 1 for
// the x passes and 0 for the columns, lengths DNSLAB_PART_LO to
// DNSLAB_PART_HI - 1 of LINE_M or LINE_N, found through DNSLAB_PART_FN.
#include "fft_line_dev.h"

namespace dnslab {
namespace {

template <typename T, int I>
LineKernel<T> pick_length(int i, int j) {
    if constexpr (I < DNSLAB_PART_HI) {
        if (i != I) return pick_length<T, I + 1>(i, j);
#if DNSLAB_PART_X
        return j ? k_line_x_inv<T, LINE_M[I]> : k_line_x_fwd<T, LINE_M[I]>;
#else
        return j == 0 ? k_line_cols<T, LINE_N[I], 0> : j == 1 ? k_line_cols<T, LINE_N[I], 1> : k_line_cols<T, LINE_N[I], 2>;
#endif
    }
    return nullptr;
}

}  // namespace

LineKernel<DNSLAB_PART_T> DNSLAB_PART_FN(int i, int j) {
    if (i < DNSLAB_PART_LO) return nullptr;
    return pick_length<DNSLAB_PART_T, DNSLAB_PART_LO>(i, j);
}

}  // namespace dnslab
