// The FFT solve of Section 2.2 in three passes over the spectrum (split y
// transform): launch interface (fft_split.hip) and the geometry both sides
// share.
#pragma once
#include "common.h"

namespace dnslab {

// One y transform of ny = R * Q is split between the x passes and the z pass:
// an x block holds the R lines y = q + Q r of one z plane, the z pass the
// remaining length-Q transforms.  The spectrum (complex, nx/2 per line: the
// kx = nx/2 column is carried inside kx = 0) is stored as rows of nx/2 values,
// row ((z * Q + q) * R + s); see fft_split.hip.
template <typename T>
struct SplitArgs {
    C2<T>* spec;
    const T* r;         // x forward: right-hand side
    T* p;               // x inverse: result
    const C2<T>* wx;    // W_m^j, j < m = nx/2
    const C2<T>* wy;    // W_ny^j
    const C2<T>* wz;    // W_nz^j
    const C2<T>* tw;    // e^{-2 pi i k / nx}, k <= m
    const double* sx2;  // sin^2(2 pi k / N)/dx^2 tables
    const double* sy2;
    const double* sz2;
    double inv_ntot;
    int nx, ny, nz;
    // x inverse of an iterate that only the immersed-boundary term reads: one
    // word per line, bit (i >> seg_lg) set where cells of that segment are read;
    // the others are not written (NULL: everything is)
    const unsigned long long* need;
    int seg_lg;
    int q;              // Q = ny / R
    int gs;             // stride of a group of R rows of the spectrum
};

// What make_split_plan chose for a grid; r == 0: the grid takes the general passes.
struct SplitPlan {
    int r, q;           // ny = r * q
    int gs;             // stride of a group of r rows of the spectrum
    int xi, ri, zi, qi; // kernel instances (indices into the length tables)
};

SplitPlan make_split_plan(int nx, int ny, int nz, int esz);

template <typename T>
hipError_t launch_split_x(const SplitArgs<T>& a, const SplitPlan& sp, bool inverse, hipStream_t s,
                          Recorder* rec = nullptr);
template <typename T>
hipError_t launch_split_z(const SplitArgs<T>& a, const SplitPlan& sp, hipStream_t s, Recorder* rec = nullptr);

// Batched replay of one recorded position (see launch_batched_stencil).
hipError_t launch_batched_split(int kind, const void* tab, const unsigned* starts, int ns, unsigned total_blocks,
                                dim3 block, size_t lds, hipStream_t s);

// The compile-time lengths: nx/2, the y factors R and Q, and nz.
constexpr int SPLIT_M[] = {16, 18, 24, 27, 32, 36, 48, 54, 64, 72, 81, 96, 108, 128, 144, 162, 192, 216, 243, 256, 288,
                           384, 512};
constexpr int SPLIT_R[] = {8, 9, 12, 16, 18};
constexpr int SPLIT_Q[] = {3, 4, 6, 8, 9, 12, 16};
constexpr int SPLIT_NZ[] = {16, 18, 24, 27, 32, 36, 48, 54, 64, 72, 81, 96, 108, 128, 144, 162, 192, 216, 256};
constexpr int SPLIT_NM = sizeof(SPLIT_M) / sizeof(int), SPLIT_NR = sizeof(SPLIT_R) / sizeof(int);
constexpr int SPLIT_NQ = sizeof(SPLIT_Q) / sizeof(int), SPLIT_NNZ = sizeof(SPLIT_NZ) / sizeof(int);

template <typename T>
using SplitKernel = void (*)(SplitArgs<T>, const BRec<SplitArgs<T>>*, const unsigned*, int);

// Kernel of an instance (defined in the fft_split_*.hip parts).
template <typename T>
SplitKernel<T> split_x_kernel(int xi, int ri, bool inverse);
template <typename T>
SplitKernel<T> split_z_kernel(int zi, int qi);

// Digits of a transform length: n = d[0] * d[1] (* d[2]).
struct SplitDigits {
    int d[3];
    int n;
};
constexpr SplitDigits split_digits(int n) {
    switch (n) {
        case 16: return {{4, 4, 1}, 2};
        case 18: return {{6, 3, 1}, 2};
        case 24: return {{6, 4, 1}, 2};
        case 27: return {{9, 3, 1}, 2};
        case 32: return {{8, 4, 1}, 2};
        case 36: return {{6, 6, 1}, 2};
        case 48: return {{8, 6, 1}, 2};
        case 54: return {{9, 6, 1}, 2};
        case 64: return {{8, 8, 1}, 2};
        case 72: return {{9, 8, 1}, 2};
        case 81: return {{9, 9, 1}, 2};
        case 96: return {{12, 8, 1}, 2};
        case 108: return {{12, 9, 1}, 2};
        case 128: return {{16, 8, 1}, 2};
        case 144: return {{12, 12, 1}, 2};
        case 162: return {{18, 9, 1}, 2};
        case 192: return {{16, 12, 1}, 2};
        case 216: return {{18, 12, 1}, 2};
        case 243: return {{9, 9, 3}, 3};
        case 256: return {{16, 16, 1}, 2};
        case 288: return {{8, 6, 6}, 3};
        case 384: return {{8, 8, 6}, 3};
        case 512: return {{8, 8, 8}, 3};
        default: return {{1, 1, 1}, 0};
    }
}

// x passes: groups of R lines per block, lines, LDS stride of one element row
// and threads.
constexpr int split_x_groups(int m) {
    return m < 24 ? 3 : m == 24 ? 4 : m < 54 ? 2 : 1;
}
constexpr int split_x_es(int lines) {
    int e = lines;
    while (e % 16 != 1) ++e;
    return e;
}
constexpr int split_x_threads(int m) { return (split_x_groups(m) * m + 63) / 64 * 64; }
#ifndef DNSLAB_SPLIT_HALF_KB
#define DNSLAB_SPLIT_HALF_KB 40
#endif
// Tiles above this exchange real and imaginary parts in turn: 512x256x192 FP64
// x passes (70 KB whole) 85 / 95 -> 82 / 81 us; smaller tiles keep the one
// barrier.
constexpr size_t SPLIT_HALF_BYTES = DNSLAB_SPLIT_HALF_KB * 1024;
constexpr size_t split_x_places(int m, int r) {   // the lines, one pad per first-digit block
    return ((size_t)m * split_x_es(split_x_groups(m) * r) + split_digits(m).d[0] + 1) / 2 * 2;
}
constexpr bool split_x_half(int m, int r, int esz) { return split_x_places(m, r) * 2 * esz > SPLIT_HALF_BYTES; }
constexpr size_t split_x_tile_bytes(int m, int r, int esz) {
    return split_x_places(m, r) * (split_x_half(m, r, esz) ? 1 : 2) * esz;
}
// The tile, then W_m and per group the factors W_ny^{q s} and W_Q^q.
constexpr size_t split_x_lds(int m, int r, int esz) {
    return split_x_tile_bytes(m, r, esz) + (size_t)(m + split_x_groups(m) * (r + 1)) * 2 * esz;
}

// z pass: a tile takes 2^lg kx columns, all z and q of one y digit, in rows of
// es places (the columns modulo a bank period, so that a wave's rows fall on
// different banks); then the tables W_nz and the z symbol.
struct SplitZGeom {
    int lg, es, nt, half;
    size_t tile, lds;
};
constexpr SplitZGeom split_z_at(int nz, int q, int esz, int lg) {
    SplitZGeom g = {lg, q << lg, 0, 0, 0, 0};
    for (int pass = 0; pass < 2; ++pass) {
        const int period = esz == 4 && g.half ? 32 : 16;
        g.es = q << lg;
        while (g.es % period != (1 << lg) % period) ++g.es;
        g.half = (size_t)nz * g.es * 2 * esz > SPLIT_HALF_BYTES;
    }
    const SplitDigits dg = split_digits(nz);
    const int dm = dg.d[0] > dg.d[1] ? dg.d[0] : dg.d[1];
    const int units = (nz > q * dm ? nz : q * dm) << lg;
    g.nt = (units + 63) / 64 * 64;
    g.tile = ((size_t)nz * g.es + 1) / 2 * 2 * (g.half ? 1 : 2) * esz;
    g.lds = g.tile + (size_t)nz * (2 * esz + 8);
    return g;
}
// The widest rows (up to 64 bytes) whose tile fits a CU and 1024 threads
// (512x256x192 FP64 z pass: rows of 16, 32, 64 bytes 277, 160, 121 us).
constexpr SplitZGeom split_z_geom(int nz, int q, int esz) {
    SplitZGeom best = split_z_at(nz, q, esz, 0);
    for (int lg = 1; (2 * esz) << lg <= 64; ++lg) {
        const SplitZGeom g = split_z_at(nz, q, esz, lg);
        if (g.lds <= 160 * 1024 && g.nt <= 1024) best = g;
    }
    return best;
}

}  // namespace dnslab
