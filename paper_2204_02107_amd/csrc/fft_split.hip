// Host side of the three-pass FFT solve: which grids take it, the tile of the
// z pass, and the launches.  The kernels are in fft_split_dev.h, compiled in
// parts (fft_split_part.hip).
#include "fft_split.h"

#include <algorithm>
#include <cstddef>

namespace dnslab {

// Instance tables of the parts: x passes and z passes by ranges of SPLIT_M and
// SPLIT_NZ; each answers NULL outside its range.
#define DNSLAB_PARTS(T, X)                        \
    SplitKernel<T> split_##X##_0(int, int, bool); \
    SplitKernel<T> split_##X##_1(int, int, bool); \
    SplitKernel<T> split_##X##_2(int, int, bool); \
    static SplitKernel<T> find_##X(int i, int j, bool inverse) {        \
        SplitKernel<T> k = split_##X##_0(i, j, inverse);                \
        if (!k) k = split_##X##_1(i, j, inverse);                       \
        return k ? k : split_##X##_2(i, j, inverse);                    \
    }
DNSLAB_PARTS(double, x64)
DNSLAB_PARTS(float, x32)
DNSLAB_PARTS(double, z64)
DNSLAB_PARTS(float, z32)
#undef DNSLAB_PARTS

template <>
SplitKernel<double> split_x_kernel<double>(int xi, int ri, bool inverse) { return find_x64(xi, ri, inverse); }
template <>
SplitKernel<float> split_x_kernel<float>(int xi, int ri, bool inverse) { return find_x32(xi, ri, inverse); }
template <>
SplitKernel<double> split_z_kernel<double>(int zi, int qi) { return find_z64(zi, qi, false); }
template <>
SplitKernel<float> split_z_kernel<float>(int zi, int qi) { return find_z32(zi, qi, false); }

namespace {

constexpr size_t LDS_MAX = 160 * 1024;
#ifndef DNSLAB_SPLIT_SMALL_CELLS
#define DNSLAB_SPLIT_SMALL_CELLS (1LL << 21)
#endif
int find(const int* t, int n, int v) {
    for (int i = 0; i < n; ++i)
        if (t[i] == v) return i;
    return -1;
}

}  // namespace

SplitPlan make_split_plan(int nx, int ny, int nz, int esz) {
    SplitPlan p = {};
    const int m = nx / 2;
    p.xi = find(SPLIT_M, SPLIT_NM, m);
    p.zi = find(SPLIT_NZ, SPLIT_NNZ, nz);
    if (nx % 2 != 0 || p.xi < 0 || p.zi < 0) return p;
    // R: small grids take the least, which gives the most and the lightest x
    // blocks (a solve of 64^3 FP64 17.1 against 20.4 us with R = 16, 192x96x64
    // 30.2 against 33.8), larger ones the greatest, which leaves the z pass
    // short columns and so wide rows (512x128x128 FP64 88 against 104 us;
    // 256x128x96 46.1 against 48.9).
    const bool small = (long long)nx * ny * nz < DNSLAB_SPLIT_SMALL_CELLS;
    for (int i = 0; i < SPLIT_NR; ++i) {
        const int ri = small ? i : SPLIT_NR - 1 - i, r = SPLIT_R[ri];
        if (ny % r != 0) continue;
        const int q = ny / r, qi = find(SPLIT_Q, SPLIT_NQ, q);
        if (qi < 0 || split_x_lds(m, r, esz) > LDS_MAX || split_z_geom(nz, q, esz).lds > LDS_MAX) continue;
        p.ri = ri;
        p.qi = qi;
        p.r = r;
        p.q = q;
        // a group of rows is padded by up to 384 bytes (what the general
        // layout's row padding leaves room for), so that the z pass, whose
        // tiles read a few values of every group, does not meet the same
        // memory channels throughout (256x128x96 FP32 38.2 -> 36.0 us)
        const int sx = (m + 1 + 15) / 16 * 16;
        p.gs = r * m + std::min(384 / (2 * esz), (sx - m) * r);
        return p;
    }
    return p;
}

template <typename T>
hipError_t launch_split_x(const SplitArgs<T>& a, const SplitPlan& sp, bool inverse, hipStream_t s, Recorder* rec) {
    const int m = SPLIT_M[sp.xi], g = split_x_groups(m);
    const int ngrp = sp.q * a.nz;
    const dim3 grid((ngrp + g - 1) / g), block(split_x_threads(m));
    const size_t lds = split_x_lds(m, sp.r, (int)sizeof(T));
    if (rec) {
        record_launch(rec, kind_code(inverse ? KK_SPLITXI : KK_SPLITXF, sp.xi * SPLIT_NR + sp.ri, sizeof(T) == 4), grid,
                      block, lds, a);
        return hipSuccess;
    }
    const SplitKernel<T> k = split_x_kernel<T>(sp.xi, sp.ri, inverse);
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, grid, block, lds, s, a, (const BRec<SplitArgs<T>>*)nullptr, (const unsigned*)nullptr, 0);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_split_z(const SplitArgs<T>& a, const SplitPlan& sp, hipStream_t s, Recorder* rec) {
    const SplitZGeom gm = split_z_geom(a.nz, sp.q, (int)sizeof(T));
    const int ntiles = ((a.nx / 2 + (1 << gm.lg) - 1) >> gm.lg) * sp.r;
    const dim3 grid(ntiles), block(gm.nt);
    const size_t lds = gm.lds;
    if (rec) {
        record_launch(rec, kind_code(KK_SPLITZ, sp.zi * SPLIT_NQ + sp.qi, sizeof(T) == 4), grid, block, lds, a);
        return hipSuccess;
    }
    const SplitKernel<T> k = split_z_kernel<T>(sp.zi, sp.qi);
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, grid, block, lds, s, a, (const BRec<SplitArgs<T>>*)nullptr, (const unsigned*)nullptr, 0);
    return hipGetLastError();
}

namespace {
template <typename T>
hipError_t split_batched(int base, int mode, const void* tab, const unsigned* st, int ns, unsigned nb, dim3 blk,
                         size_t lds, hipStream_t s) {
    const SplitKernel<T> k = base == KK_SPLITZ ? split_z_kernel<T>(mode / SPLIT_NQ, mode % SPLIT_NQ)
                                               : split_x_kernel<T>(mode / SPLIT_NR, mode % SPLIT_NR, base == KK_SPLITXI);
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3(nb), blk, lds, s, SplitArgs<T>{}, (const BRec<SplitArgs<T>>*)tab, st, ns);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_batched_split(int kind, const void* tab, const unsigned* st, int ns, unsigned nb, dim3 blk,
                                size_t lds, hipStream_t s) {
    const int base = kind >> 12, mode = (kind >> 1) & 2047;
    return (kind & 1) ? split_batched<float>(base, mode, tab, st, ns, nb, blk, lds, s)
                      : split_batched<double>(base, mode, tab, st, ns, nb, blk, lds, s);
}

template hipError_t launch_split_x<double>(const SplitArgs<double>&, const SplitPlan&, bool, hipStream_t, Recorder*);
template hipError_t launch_split_x<float>(const SplitArgs<float>&, const SplitPlan&, bool, hipStream_t, Recorder*);
template hipError_t launch_split_z<double>(const SplitArgs<double>&, const SplitPlan&, hipStream_t, Recorder*);
template hipError_t launch_split_z<float>(const SplitArgs<float>&, const SplitPlan&, hipStream_t, Recorder*);

}  // namespace dnslab
