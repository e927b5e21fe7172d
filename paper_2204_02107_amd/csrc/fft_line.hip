// Host side of the axis-by-axis FFT solve on register tiles: which grids take
// it, and the launches.  The kernels are in fft_line_dev.h, compiled in parts
// (fft_line_part.hip).
#include "fft_line.h"

#include <algorithm>
#include <cstddef>

namespace dnslab {

// Instance tables of the parts, by ranges of LINE_M and LINE_N; each answers
// NULL outside its range (j: inverse for the x passes, the mode for columns).
#define DNSLAB_PARTS(T, X)                        \
    LineKernel<T> line_##X##_0(int, int);         \
    LineKernel<T> line_##X##_1(int, int);         \
    static LineKernel<T> find_##X(int i, int j) { \
        const LineKernel<T> k = line_##X##_0(i, j); \
        return k ? k : line_##X##_1(i, j);        \
    }
DNSLAB_PARTS(double, x64)
DNSLAB_PARTS(float, x32)
DNSLAB_PARTS(double, c64)
DNSLAB_PARTS(float, c32)
#undef DNSLAB_PARTS

template <>
LineKernel<double> line_x_kernel<double>(int xi, bool inverse) { return find_x64(xi, inverse); }
template <>
LineKernel<float> line_x_kernel<float>(int xi, bool inverse) { return find_x32(xi, inverse); }
template <>
LineKernel<double> line_cols_kernel<double>(int ci, int mode) { return find_c64(ci, mode); }
template <>
LineKernel<float> line_cols_kernel<float>(int ci, int mode) { return find_c32(ci, mode); }

namespace {
int find(const int* t, int n, int v) {
    for (int i = 0; i < n; ++i)
        if (t[i] == v) return i;
    return -1;
}
}  // namespace

LinePlan make_line_plan(int nx, int ny, int nz) {
    LinePlan p = {};
    p.xi = nx % 2 == 0 ? find(LINE_M, LINE_NM, nx / 2) : -1;
    p.yi = find(LINE_N, LINE_NN, ny);
    p.zi = nz == 1 ? 0 : find(LINE_N, LINE_NN, nz);
    p.on = p.xi >= 0 && p.yi >= 0 && p.zi >= 0;
    return p;
}

template <typename T>
hipError_t launch_line_x(const LineArgs<T>& a, int xi, bool inverse, hipStream_t s, Recorder* rec) {
    const LineGeom gm = line_x_geom(LINE_M[xi], (int)sizeof(T));
    const dim3 grid((a.nlines + gm.nl - 1) / gm.nl), block(gm.nt);
    if (rec) {
        record_launch(rec, kind_code(inverse ? KK_LINEXI : KK_LINEXF, xi, sizeof(T) == 4), grid, block, gm.lds, a);
        return hipSuccess;
    }
    const LineKernel<T> k = line_x_kernel<T>(xi, inverse);
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, grid, block, gm.lds, s, a, (const BRec<LineArgs<T>>*)nullptr, (const unsigned*)nullptr, 0);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_line_cols(const LineArgs<T>& a, int ci, int mode, hipStream_t s, Recorder* rec) {
    const LineGeom gm = line_c_geom(LINE_N[ci], (int)sizeof(T));
    const dim3 grid((unsigned)((a.nx / 2 + gm.nl - 1) / gm.nl) * a.nplanes), block(gm.nt);
    if (rec) {
        record_launch(rec, kind_code(KK_LINEC, ci * 3 + mode, sizeof(T) == 4), grid, block, gm.lds, a);
        return hipSuccess;
    }
    const LineKernel<T> k = line_cols_kernel<T>(ci, mode);
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, grid, block, gm.lds, s, a, (const BRec<LineArgs<T>>*)nullptr, (const unsigned*)nullptr, 0);
    return hipGetLastError();
}

namespace {
template <typename T>
hipError_t line_batched(int base, int mode, const void* tab, const unsigned* st, int ns, unsigned nb, dim3 blk,
                        size_t lds, hipStream_t s) {
    const LineKernel<T> k =
        base == KK_LINEC ? line_cols_kernel<T>(mode / 3, mode % 3) : line_x_kernel<T>(mode, base == KK_LINEXI);
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3(nb), blk, lds, s, LineArgs<T>{}, (const BRec<LineArgs<T>>*)tab, st, ns);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_batched_line(int kind, const void* tab, const unsigned* st, int ns, unsigned nb, dim3 blk,
                               size_t lds, hipStream_t s) {
    const int base = kind >> 12, mode = (kind >> 1) & 2047;
    return (kind & 1) ? line_batched<float>(base, mode, tab, st, ns, nb, blk, lds, s)
                      : line_batched<double>(base, mode, tab, st, ns, nb, blk, lds, s);
}

template hipError_t launch_line_x<double>(const LineArgs<double>&, int, bool, hipStream_t, Recorder*);
template hipError_t launch_line_x<float>(const LineArgs<float>&, int, bool, hipStream_t, Recorder*);
template hipError_t launch_line_cols<double>(const LineArgs<double>&, int, int, hipStream_t, Recorder*);
template hipError_t launch_line_cols<float>(const LineArgs<float>&, int, int, hipStream_t, Recorder*);

}  // namespace dnslab
