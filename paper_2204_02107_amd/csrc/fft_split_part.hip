// One part of the kernel instances of the three-pass FFT solve, so that the
// parts compile side by side: DNSLAB_PART_T the real type, DNSLAB_PART_X 1 for
// the x passes and 0 for the z pass, lengths DNSLAB_PART_LO to DNSLAB_PART_HI - 1
// of SPLIT_M or SPLIT_NZ, found through the function DNSLAB_PART_FN.
#include "fft_split_dev.h"

namespace dnslab {
namespace {

template <typename T, int I, int J>
SplitKernel<T> pick(int j, bool inverse) {
#if DNSLAB_PART_X
    if constexpr (J < SPLIT_NR) {
        if (j != J) return pick<T, I, J + 1>(j, inverse);
        return inverse ? k_split_x_inv<T, SPLIT_M[I], SPLIT_R[J]> : k_split_x_fwd<T, SPLIT_M[I], SPLIT_R[J]>;
    }
#else
    if constexpr (J < SPLIT_NQ) {
        if (j != J) return pick<T, I, J + 1>(j, inverse);
        return k_split_z<T, SPLIT_NZ[I], SPLIT_Q[J]>;
    }
#endif
    return nullptr;
}
template <typename T, int I>
SplitKernel<T> pick_length(int i, int j, bool inverse) {
    if constexpr (I < DNSLAB_PART_HI) {
        if (i != I) return pick_length<T, I + 1>(i, j, inverse);
        return pick<T, I, 0>(j, inverse);
    }
    return nullptr;
}

}  // namespace

SplitKernel<DNSLAB_PART_T> DNSLAB_PART_FN(int i, int j, bool inverse) {
    if (i < DNSLAB_PART_LO) return nullptr;
    return pick_length<DNSLAB_PART_T, DNSLAB_PART_LO>(i, j, inverse);
}

}  // namespace dnslab
