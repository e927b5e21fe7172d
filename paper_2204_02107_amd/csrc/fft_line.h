// The FFT solve of Section 2.2 axis by axis, on tiles kept in registers: launch
// interface (fft_line.hip) and the geometry both sides share.  For grids whose
// y transform is too long to be split between the x and z passes
// (fft_split.h), five passes: x, y, z with the divide, y, x; for 2D grids
// (nz = 1) three: x, y with the divide, x.
//
// Against the general passes (one solve): 1024x512x256 FP64 2264 -> 2004 us (x
// forward 406 -> 378, y 449 -> 396, z 510 -> 429, x inverse 453 -> 405: 5.0 to
// 5.7 TB/s), FP32 1220 -> 1080; 1536x192 FP64 42 -> 18 us (five launches to
// three, each bound by its own start and drain).  What bounds the large grid is
// HBM; the passes are 10 to 15% short of what a copy kernel reaches.
#pragma once
#include "common.h"
#include "fft_split.h"

namespace dnslab {

// Spectrum: rows of rs complex values (nx/2 used, the kx = nx/2 column inside
// kx = 0 as in fft_split_dev.h), row (y or ky place) + ny * z.
template <typename T>
struct LineArgs {
    C2<T>* spec;
    const T* r;         // x forward: right-hand side
    T* p;               // x inverse: result
    const C2<T>* wx;    // W_m^j, j < m = nx/2
    const C2<T>* wc;    // W_n^j of the columns (y or z)
    const C2<T>* tw;    // e^{-2 pi i k / nx}, k <= m
    const double* sx2;  // symbol tables: kx, the columns' frequency, the planes'
    const double* sc2;
    const double* sp2;
    double inv_ntot;
    const unsigned long long* need;   // as SplitArgs::need
    int seg_lg;
    int nx;
    int nlines;         // x passes: lines
    int rs;             // row stride
    int rstr, pstr;     // column passes: strides of consecutive rows of a column and of planes
    int nplanes;
    int d0, d1, np;     // digits of the planes' axis, whose frequencies lie in digit order (np = 0: in order)
};

struct LinePlan {
    int on;
    int xi, yi, zi;     // kernel instances (zi unused for nz = 1)
};

LinePlan make_line_plan(int nx, int ny, int nz);

template <typename T>
hipError_t launch_line_x(const LineArgs<T>& a, int xi, bool inverse, hipStream_t s, Recorder* rec = nullptr);
// mode 0: forward, 1: inverse, 2: forward, divide, inverse.
template <typename T>
hipError_t launch_line_cols(const LineArgs<T>& a, int ci, int mode, hipStream_t s, Recorder* rec = nullptr);

hipError_t launch_batched_line(int kind, const void* tab, const unsigned* starts, int ns, unsigned total_blocks,
                               dim3 block, size_t lds, hipStream_t s);

constexpr int LINE_M[] = {162, 192, 216, 243, 256, 288, 324, 384, 432, 486, 512, 576, 648, 729, 768, 864, 972, 1024,
                          1152, 1296, 1458, 1536, 1728};
constexpr int LINE_N[] = {54, 64, 72, 81, 96, 108, 128, 144, 162, 192, 216, 243, 256, 288, 324, 384, 432, 512};
constexpr int LINE_NM = sizeof(LINE_M) / sizeof(int), LINE_NN = sizeof(LINE_N) / sizeof(int);

template <typename T>
using LineKernel = void (*)(LineArgs<T>, const BRec<LineArgs<T>>*, const unsigned*, int);
template <typename T>
LineKernel<T> line_x_kernel(int xi, bool inverse);
template <typename T>
LineKernel<T> line_cols_kernel(int ci, int mode);

constexpr SplitDigits line_digits(int n) {
    switch (n) {
        case 288: return {{18, 16, 1}, 2};
        case 324: return {{18, 18, 1}, 2};
        case 384: return {{8, 8, 6}, 3};
        case 432: return {{12, 6, 6}, 3};
        case 486: return {{9, 9, 6}, 3};
        case 512: return {{8, 8, 8}, 3};
        case 576: return {{9, 8, 8}, 3};
        case 648: return {{9, 9, 8}, 3};
        case 729: return {{9, 9, 9}, 3};
        case 768: return {{12, 8, 8}, 3};
        case 864: return {{12, 9, 8}, 3};
        case 972: return {{12, 9, 9}, 3};
        case 1024: return {{16, 8, 8}, 3};
        case 1152: return {{12, 12, 8}, 3};
        case 1296: return {{12, 12, 9}, 3};
        case 1458: return {{18, 9, 9}, 3};
        case 1536: return {{16, 12, 8}, 3};
        case 1728: return {{12, 12, 12}, 3};
        default: return split_digits(n);
    }
}

// A tile: n places of nl lines (place p of line l at p * nl + p / S0 * pad + l),
// nt threads.
struct LineGeom {
    int nl, nt, half, pad, wlds;
    size_t tile, lds;
};
constexpr LineGeom line_geom(int n, int nl, int esz, int pad, int wlds) {
    LineGeom g = {nl, 0, 0, pad, wlds, 0, 0};
    const SplitDigits dg = line_digits(n);
    int units = 0;
    for (int i = 0; i < dg.n; ++i) units = nl * (n / dg.d[i]) > units ? nl * (n / dg.d[i]) : units;
    g.nt = (units + 63) / 64 * 64;
    if (g.nt > 1024) g.nt = 1024;
    const size_t places = ((size_t)n * nl + (size_t)dg.d[0] * pad + 1) / 2 * 2;
    g.half = places * 2 * esz > SPLIT_HALF_BYTES;
    g.tile = places * (g.half ? 1 : 2) * esz;
    g.lds = g.tile + (wlds ? (size_t)n * 2 * esz : 0);
    return g;
}
// x passes: lines per block, so that a block has 64 to 256 threads; a pad of
// one spreads consecutive frequencies, S0 places apart, over the banks.  W_m
// stays in global memory: a copy in LDS takes a third of a block's and with it
// a third of the blocks per CU (1024x512x256, x inverse 461 -> 405 us FP64,
// 267 -> 238 us FP32; x forward 377 and 225 us either way).
constexpr LineGeom line_x_geom(int m, int esz) {
    return line_geom(m, m >= 768 ? 1 : m >= 384 ? 2 : 4, esz, 1, 0);
}
// Column passes: row segments of 128 bytes; the pad keeps the last digit's
// units, S0 places apart, off each other's banks.  W_n in LDS, read by several
// rows' worth of lanes each (in global memory FP32 y 180 -> 221 us, z 228 ->
// 275 us on 1024x512x256).
constexpr LineGeom line_c_geom(int n, int esz) { return line_geom(n, 64 / esz, esz, 64 / esz, 1); }

}  // namespace dnslab
