// Kernels of the three-pass FFT solve (fft_split.hip), as templates that the
// fft_split_*.hip parts instantiate.
//
// The pressure equation is diagonal in Fourier space.  Instead of five passes
// over the half spectrum (x, y, z with the divide, y, x), the y transform is
// split by the Cooley-Tukey step, ny = R Q, y = q + Q r, ky = s + R t:
//
//   Y[s + R t] = sum_q W_Q^{q t} W_ny^{q s} sum_r y[q + Q r] W_R^{r s},
//
// the inner sums being done by the x passes, whose blocks hold the R lines
// q + Q r of a z plane, and the outer ones by the z pass, whose blocks hold all
// (z, q) of one s for a few kx.  A solve then reads and writes the spectrum
// three times instead of five, in three launches.
//
// A block keeps its tile in registers, one digit of the transform per thread,
// and exchanges it through LDS between the digits.  The exchanges work in
// place (decimation in frequency forward, in time on the way back): a thread
// writes the places it read, so an exchange needs one barrier, and frequencies
// stay in digit order, which the last addresses take into account.  Large
// tiles exchange the real parts, then the imaginary parts, through half the
// LDS (three barriers), so that two or more blocks share a CU and one
// transforms while another loads or stores.  The outermost digit of each pass
// (R or Q) is transformed between the global accesses and the first or last
// exchange.
//
// The real transform packs x pairs: Z = FFT_m(x_even + i x_odd).  The y digit
// is transformed first, on Z: sum_r conj Z_r[m-k] W^{rs} is the conjugate of
// the transform at -s, so X[k] at digit s comes from Z[k] at s and Z[m-k] at
// -s.  The factors f^s, f = W_ny^q, are applied with the y digit, on Z: Z[k] at
// s then carries f^s and Z[m-k] at -s carries f^{R-s}, so its conjugate lacks
// f^R = W_Q^q (for s > 0).  X[0] and X[m] (the Nyquist column) are real
// combinations of Re Z[0] and Im Z[0], and the symbol of central differences, -sum sin^2(2 pi k/N)/dx^2,
// is the same at kx = 0 and kx = m and even in (ky, kz): the solve maps Re
// Z[0] and Im Z[0] separately by one real operator, so the column kx = 0 holds
// Z[0] itself and the Nyquist column needs no storage.
//
// Measured (one solve, against the five passes; 64^3, 192x96x64 and the FP32
// 256x128x96 against the fused y/z plane pass they took before):
//   FP64: 64^3 29 -> 17 us, 216x108x72 104 -> 33, 256x128x96 67 -> 46,
//         512x256x192 402 -> 297;  FP32: 512x256x192 245 -> 170.
// On 512x256x192 FP64 the x passes move 4.8 to 4.9 TB/s, the z pass 3.5: its
// blocks of 1024 threads and 104 KB run one to a CU, so that its exchanges
// (about 40 us of it) are not hidden behind its loads and stores.  The same
// pass with rows of 32 bytes (52 KB tiles) took 160 us instead of 121: short
// rows at power-of-two strides cost more than the second block gains.
#pragma once

#include <type_traits>

#include "fft_dev.h"
#include "fft_split.h"

namespace dnslab {
namespace {

template <typename T>
__device__ __forceinline__ bool split_args(SplitArgs<T>& a, unsigned& blk, unsigned& nb,
                                           const BRec<SplitArgs<T>>* tab, const unsigned* st, int ns) {
    blk = blockIdx.x;
    nb = gridDim.x;
    if (tab) {
        const int e = batch_slot(st, ns);
        blk -= st[e];
        nb = tab[e].g[0];
        a = tab[e].a;
        return true;
    }
    return false;
}

// Global accesses.  The argument block may come from the batched table, where
// the compiler cannot tell that its pointers are global: it would use flat
// accesses, which count with the LDS operations and hold up every LDS wait.
template <typename T>
using V2 = T __attribute__((ext_vector_type(2)));
template <typename T>
__device__ __forceinline__ C2<T> ldg(const C2<T>* base, unsigned i) {
    const V2<T> v = ((const __attribute__((address_space(1))) V2<T>*)base)[i];
    return C2<T>{v.x, v.y};
}
template <typename T>
__device__ __forceinline__ void stg(C2<T>* base, unsigned i, C2<T> v) {
    ((__attribute__((address_space(1))) V2<T>*)base)[i] = V2<T>{v.x, v.y};
}
__device__ __forceinline__ double ldg(const double* base, unsigned i) {
    return ((const __attribute__((address_space(1))) double*)base)[i];
}

__device__ __forceinline__ unsigned long long need_word(const unsigned long long* need, int line) {
    return ((const __attribute__((address_space(1))) unsigned long long*)need)[line];
}

// Barrier between LDS stages that waits for the wave's LDS operations only:
// global loads of the next tile and stores of the last one stay in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// A stage: units u < N of D values each at places base(u) + r * S.
template <int N_, int D_, int S_>
struct Stage {
    static constexpr int N = N_, D = D_, S = S_;
};
template <class St, int NT>
constexpr int nunits() { return (St::N + NT - 1) / NT; }
// Which part of the complex values an access moves.
enum Part { RE = 0, IM = 1, BOTH = 2 };

template <int P, typename T>
__device__ __forceinline__ void put(C2<T>* s, int e, const C2<T>& v) {
    if constexpr (P == BOTH) s[e] = v;
    else reinterpret_cast<T*>(s)[e] = P == RE ? v.x : v.y;
}
template <int P, typename T>
__device__ __forceinline__ void get(const C2<T>* s, int e, C2<T>& v) {
    if constexpr (P == BOTH) v = s[e];
    else if constexpr (P == RE) v.x = reinterpret_cast<const T*>(s)[e];
    else v.y = reinterpret_cast<const T*>(s)[e];
}
template <class St, int NT, int P, typename T, class Base>
__device__ __forceinline__ void put_stage(C2<T>* s, const C2<T> (&v)[nunits<St, NT>()][St::D], int tid, Base base) {
#pragma unroll
    for (int i = 0; i < nunits<St, NT>(); ++i)
        if (tid + i * NT < St::N) {
            const int e = base(tid + i * NT);
#pragma unroll
            for (int r = 0; r < St::D; ++r) put<P>(s, e + r * St::S, v[i][r]);
        }
}
template <class St, int NT, int P, typename T, class Base>
__device__ __forceinline__ void get_stage(const C2<T>* s, C2<T> (&v)[nunits<St, NT>()][St::D], int tid, Base base) {
#pragma unroll
    for (int i = 0; i < nunits<St, NT>(); ++i)
        if (tid + i * NT < St::N) {
            const int e = base(tid + i * NT);
#pragma unroll
            for (int r = 0; r < St::D; ++r) get<P>(s, e + r * St::S, v[i][r]);
        }
}
// One exchange: puts(part), barrier, gets(part); HALF: the real parts, then
// the imaginary ones, in the same places.
template <bool HALF, class Put, class Get>
__device__ __forceinline__ void exchange(Put puts, Get gets) {
    if constexpr (HALF) {
        puts(std::integral_constant<int, RE>{});
        lds_barrier();
        gets(std::integral_constant<int, RE>{});
        lds_barrier();
        puts(std::integral_constant<int, IM>{});
        lds_barrier();
        gets(std::integral_constant<int, IM>{});
    } else {
        puts(std::integral_constant<int, BOTH>{});
        lds_barrier();
        gets(std::integral_constant<int, BOTH>{});
    }
}
// Exchange between two stages of values in registers.
template <bool HALF, int NT, class A, class B, typename T, class BA, class BB>
__device__ __forceinline__ void exchange_stages(C2<T>* s, const C2<T> (&v)[nunits<A, NT>()][A::D],
                                                C2<T> (&w)[nunits<B, NT>()][B::D], int tid, BA ba, BB bb) {
    exchange<HALF>([&](auto p) { put_stage<A, NT, decltype(p)::value>(s, v, tid, ba); },
                   [&](auto p) { get_stage<B, NT, decltype(p)::value>(s, w, tid, bb); });
}

// Geometry of the x passes.  Place p of line l lies at p * ES + p / S0 + l (the
// pad per first-digit block spreads consecutive frequencies, S0 rows apart,
// over the banks).
template <typename T, int M, int R>
struct XG {
    static constexpr SplitDigits dg = split_digits(M);
    static constexpr int G = split_x_groups(M), NL = G * R, ES = split_x_es(NL), NT = split_x_threads(M);
    static constexpr int D0 = dg.d[0], D1 = dg.d[1], D2 = dg.d[2];
    static constexpr int S0 = M / D0, S1 = S0 / D1;
    static constexpr bool HALF = split_x_half(M, R, (int)sizeof(T));
    using Io = Stage<G * M, R, 1>;                          // unit (g, n): the R lines of a group
    using F0 = Stage<NL * (M / D0), D0, S0 * ES + 1>;       // digit i: unit (line, t)
    using F1 = Stage<NL * (M / D1), D1, S1 * ES>;
    using F2 = Stage<NL * (M / D2), D2, ES>;                // (three digits: stride 1)
    static constexpr int H = (M + 1) / 2, ITEMS = NL * H, NI = (ITEMS + NT - 1) / NT;   // pairs (k, m - k) of the lines
    static_assert(nunits<Io, NT>() == 1 && G * (R + 1) <= NT, "one line position and one factor per thread");

    static __device__ __forceinline__ int io(int u) {
        const int g = u / M, n = u % M;
        return n * ES + n / S0 + g * R;
    }
    template <int S, int L>
    static __device__ __forceinline__ int digit(int u) {
        const int l = u % NL, t = u / NL, p = (t / S) * L + t % S;
        return p * ES + p / S0 + l;
    }
    static __device__ __forceinline__ int f0(int u) { return digit<S0, M>(u); }
    static __device__ __forceinline__ int f1(int u) { return digit<S1, S0>(u); }
    static __device__ __forceinline__ int f2(int u) { return digit<1, S1>(u); }
    // row offset of frequency k
    static __device__ __forceinline__ int freq(int k) {
        const int k0 = k % D0, h = k / D0, k1 = h % D1, k2 = h / D1;
        return (k0 * S0 + k1 * S1 + k2) * ES + k0;
    }
};

// Transform of a digit (stride S in blocks of L places) of every unit, with
// its twiddles W_L^{k j} after (forward) or before (inverse) it.
template <class X, int M, int S, bool INV, class Tab, typename T, int U, int D>
__device__ __forceinline__ void x_digit(C2<T> (&v)[U][D], const Tab& W, int tid) {
    constexpr int L = D * S;
#pragma unroll
    for (int i = 0; i < U; ++i) {
        const int j = ((tid + i * X::NT) / X::NL) % S;
        if (INV && S > 1) {
#pragma unroll
            for (int r = 1; r < D; ++r) v[i][r] = cmulc(v[i][r], W[r * j * (M / L)]);
        }
        DFT<T, D, INV>::run(v[i]);
        if (!INV && S > 1) {
#pragma unroll
            for (int r = 1; r < D; ++r) v[i][r] = cmul(v[i][r], W[r * j * (M / L)]);
        }
    }
}

// One pair of frequencies of a line: (k at s, m - k at -s); k = 0 stands for
// kx = 0, which passes as it is, and, m even, kx = m/2, where X = conj Z (m
// odd: two is false, there is nothing to pair with).
template <class X, int M, int R>
struct XItem {
    int g, sd, k, kb, l, lm;
    unsigned pa, pb;     // places in the spectrum
    bool on, two;
    __device__ __forceinline__ XItem(int it, int blk, int ngrp, int gs) {
        l = it / X::H;
        k = it - l * X::H;
        g = l / R;
        sd = l - g * R;
        const int grp = blk * X::G + g, sm = (R - sd) % R;
        lm = g * R + sm;
        kb = k ? M - k : M / 2;
        two = M % 2 == 0 || k != 0;
        on = it < X::ITEMS && grp < ngrp;
        pa = (unsigned)(grp * gs + sd * M + k);
        pb = (unsigned)(grp * gs + (k ? sm : sd) * M + kb);
    }
};

// The lines' factors W_ny^{q s} (thread g R + s) and W_Q^q (thread NL + g).
template <class X, int R, typename T>
__device__ __forceinline__ C2<T> x_factor(const SplitArgs<T>& a, int blk, int tid) {
    if (tid >= X::G * (R + 1)) return C2<T>{T(0), T(0)};
    const int g = tid < X::NL ? tid / R : tid - X::NL, q = (blk * X::G + g) % a.q;
    return ldg(a.wy, tid < X::NL ? q * (tid - g * R) : q * R);
}

template <typename T, int M, int R>
__global__ __launch_bounds__(split_x_threads(M)) void k_split_x_fwd(SplitArgs<T> a, const BRec<SplitArgs<T>>* tab,
                                                                    const unsigned* st, int ns) {
    using X = XG<T, M, R>;
    constexpr int NT = X::NT, NI = X::NI;
    extern __shared__ unsigned char smem_raw[];
    C2<T>* s = reinterpret_cast<C2<T>*>(smem_raw);
    C2<T>* W = reinterpret_cast<C2<T>*>(smem_raw + split_x_tile_bytes(M, R, (int)sizeof(T)));
    C2<T>* wy = W + M;
    unsigned blk, nb;
    split_args(a, blk, nb, tab, st, ns);
    const int tid = threadIdx.x, Q = a.q, ngrp = Q * a.nz;
    const C2<T> wy0 = x_factor<X, R>(a, (int)blk, tid);
    C2<T> v0[1][R];
    const int g0 = tid / M, n0 = tid % M, grp0 = (int)blk * X::G + g0;
#pragma unroll
    for (int r = 0; r < R; ++r) v0[0][r] = C2<T>{T(0), T(0)};
    if (tid < X::Io::N && grp0 < ngrp) {
        const int z = grp0 / Q, q = grp0 - z * Q;
        // (rows of M complex values; every offset fits 32 bits at the compiled
        // lengths)
        const C2<T>* src = reinterpret_cast<const C2<T>*>(a.r);
        const unsigned o = (unsigned)(z * a.ny + q) * M + n0, dl = (unsigned)Q * M;
#pragma unroll
        for (int r = 0; r < R; ++r) v0[0][r] = ldg(src + r * dl, o);
    }
    for (int j = tid; j < M; j += NT) W[j] = ldg(a.wx, j);
    if (tid < X::G * (R + 1)) wy[tid] = wy0;
    lds_barrier();
    DFT<T, R, false>::run(v0[0]);
    if (tid < X::Io::N) {
#pragma unroll
        for (int r = 1; r < R; ++r) v0[0][r] = cmul(v0[0][r], wy[g0 * R + r]);
    }
    C2<T> v1[nunits<typename X::F0, NT>()][X::D0], v2[nunits<typename X::F1, NT>()][X::D1];
    exchange_stages<X::HALF, NT, typename X::Io, typename X::F0>(s, v0, v1, tid, X::io, X::f0);
    x_digit<X, M, X::S0, false>(v1, W, tid);
    exchange_stages<X::HALF, NT, typename X::F0, typename X::F1>(s, v1, v2, tid, X::f0, X::f1);
    x_digit<X, M, X::S1, false>(v2, W, tid);
    C2<T> za[NI], zb[NI];
    auto gets = [&](auto p) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const XItem<X, M, R> q(tid + i * NT, (int)blk, ngrp, a.gs);
            if (tid + i * NT < X::ITEMS) {
                get<decltype(p)::value>(s, X::freq(q.k) + q.l, za[i]);
                if (q.two) get<decltype(p)::value>(s, X::freq(q.kb) + q.lm, zb[i]);
            }
        }
    };
    if constexpr (X::dg.n == 3) {
        C2<T> v3[nunits<typename X::F2, NT>()][X::D2];
        exchange_stages<X::HALF, NT, typename X::F1, typename X::F2>(s, v2, v3, tid, X::f1, X::f2);
        x_digit<X, M, 1, false>(v3, W, tid);
        exchange<X::HALF>([&](auto p) { put_stage<typename X::F2, NT, decltype(p)::value>(s, v3, tid, X::f2); }, gets);
    } else {
        exchange<X::HALF>([&](auto p) { put_stage<typename X::F1, NT, decltype(p)::value>(s, v2, tid, X::f1); }, gets);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const XItem<X, M, R> q(tid + i * NT, (int)blk, ngrp, a.gs);
        if (!q.on) continue;
        const C2<T> fr = q.sd ? wy[X::NL + q.g] : C2<T>{T(1), T(0)};
        const C2<T> zr = cmulc(zb[i], fr);
        const C2<T> w = ldg(a.tw, q.k), wm = C2<T>{-w.x, w.y};
        stg(a.spec, q.pa, q.k ? r2c_post(za[i], zr, w) : za[i]);
        if (q.two) stg(a.spec, q.pb, q.k ? cmul(r2c_post(zr, za[i], wm), fr) : conj_(zr));
    }
}

template <typename T, int M, int R>
__global__ __launch_bounds__(split_x_threads(M)) void k_split_x_inv(SplitArgs<T> a, const BRec<SplitArgs<T>>* tab,
                                                                    const unsigned* st, int ns) {
    using X = XG<T, M, R>;
    constexpr int NT = X::NT, NI = X::NI;
    extern __shared__ unsigned char smem_raw[];
    C2<T>* s = reinterpret_cast<C2<T>*>(smem_raw);
    C2<T>* W = reinterpret_cast<C2<T>*>(smem_raw + split_x_tile_bytes(M, R, (int)sizeof(T)));
    C2<T>* wy = W + M;
    unsigned blk, nb;
    split_args(a, blk, nb, tab, st, ns);
    const int tid = threadIdx.x, Q = a.q, ngrp = Q * a.nz;
    const C2<T> wy0 = x_factor<X, R>(a, (int)blk, tid);
    C2<T> xa[NI], xb[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const XItem<X, M, R> q(tid + i * NT, (int)blk, ngrp, a.gs);
        xa[i] = xb[i] = C2<T>{T(0), T(0)};
        if (q.on) {
            xa[i] = ldg(a.spec, q.pa);
            if (q.two) xb[i] = ldg(a.spec, q.pb);
        }
    }
    for (int j = tid; j < M; j += NT) W[j] = ldg(a.wx, j);
    if (tid < X::G * (R + 1)) wy[tid] = wy0;
    lds_barrier();
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const XItem<X, M, R> q(tid + i * NT, (int)blk, ngrp, a.gs);
        if (!q.on) continue;
        const C2<T> fr = q.sd ? wy[X::NL + q.g] : C2<T>{T(1), T(0)};
        const C2<T> w = ldg(a.tw, q.k), wm = C2<T>{-w.x, w.y};
        const C2<T> x = xa[i], xr = cmulc(xb[i], fr);
        const C2<T> c2 = conj_(cmulc(xb[i], fr));
        if (q.k) {
            xa[i] = c2r_pre(x, xr, w);
            xb[i] = cmul(c2r_pre(xr, x, wm), fr);
        } else {
            xa[i] = cadd(x, x);
            xb[i] = cadd(c2, c2);
        }
    }
    auto puts = [&](auto p) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const XItem<X, M, R> q(tid + i * NT, (int)blk, ngrp, a.gs);
            if (tid + i * NT < X::ITEMS) {
                put<decltype(p)::value>(s, X::freq(q.k) + q.l, xa[i]);
                if (q.two) put<decltype(p)::value>(s, X::freq(q.kb) + q.lm, xb[i]);
            }
        }
    };
    C2<T> v0[1][R], v1[nunits<typename X::F0, NT>()][X::D0], v2[nunits<typename X::F1, NT>()][X::D1];
    if constexpr (X::dg.n == 3) {
        C2<T> v3[nunits<typename X::F2, NT>()][X::D2];
        exchange<X::HALF>(puts, [&](auto p) { get_stage<typename X::F2, NT, decltype(p)::value>(s, v3, tid, X::f2); });
        x_digit<X, M, 1, true>(v3, W, tid);
        exchange_stages<X::HALF, NT, typename X::F2, typename X::F1>(s, v3, v2, tid, X::f2, X::f1);
    } else {
        exchange<X::HALF>(puts, [&](auto p) { get_stage<typename X::F1, NT, decltype(p)::value>(s, v2, tid, X::f1); });
    }
    x_digit<X, M, X::S1, true>(v2, W, tid);
    exchange_stages<X::HALF, NT, typename X::F1, typename X::F0>(s, v2, v1, tid, X::f1, X::f0);
    x_digit<X, M, X::S0, true>(v1, W, tid);
    exchange_stages<X::HALF, NT, typename X::F0, typename X::Io>(s, v1, v0, tid, X::f0, X::io);
    const int g0 = X::G == 1 ? 0 : tid / M, n0 = tid - g0 * M, grp0 = (int)blk * X::G + g0;
    if (tid < X::Io::N && grp0 < ngrp) {
#pragma unroll
        for (int r = 1; r < R; ++r) v0[0][r] = cmulc(v0[0][r], wy[g0 * R + r]);
        DFT<T, R, true>::run(v0[0]);
        const int z = grp0 / Q, q = grp0 - z * Q;
        C2<T>* dst = reinterpret_cast<C2<T>*>(a.p);
        const int line = z * a.ny + q;
        const unsigned o = (unsigned)line * M + n0, dl = (unsigned)Q * M;
        if (a.need) {
            const unsigned seg = (unsigned)(2 * n0) >> a.seg_lg;
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (need_word(a.need, line + Q * r) >> seg & 1u) stg(dst + r * dl, o, v0[0][r]);
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) stg(dst + r * dl, o, v0[0][r]);
        }
    }
}

// z pass: the tile of one y digit s and TX consecutive kx, all z and q; (z, q or
// t, c) at place z * ES + q * TX + c.
template <typename T, int NZ, int Q>
__global__ __launch_bounds__(split_z_geom(NZ, Q, (int)sizeof(T)).nt) void k_split_z(SplitArgs<T> a,
                                                                                 const BRec<SplitArgs<T>>* tab,
                                                                                 const unsigned* st, int ns) {
    constexpr SplitDigits dg = split_digits(NZ);
    constexpr SplitZGeom gm = split_z_geom(NZ, Q, (int)sizeof(T));
    constexpr int D0 = dg.d[0], D1 = dg.d[1], NT = gm.nt, ES = gm.es, LG = gm.lg, TX = 1 << LG, LT = Q * TX;
    constexpr bool HALF = gm.half != 0;
    using Io = Stage<NZ * TX, Q, TX>;          // unit (z, c): all q or t
    using Z0 = Stage<LT * D1, D0, D1 * ES>;    // unit (j, line): z = j + D1 r, or k0 = r
    using Z1 = Stage<LT * D0, D1, ES>;         // unit (k0, line): j = r, or kz = k0 + D0 r
    extern __shared__ unsigned char smem_raw[];
    C2<T>* sm = reinterpret_cast<C2<T>*>(smem_raw);
    C2<T>* wz = reinterpret_cast<C2<T>*>(smem_raw + gm.tile);
    double* sz2 = reinterpret_cast<double*>(wz + NZ);
    unsigned blk, nb;
    // neighbouring kx tiles share the 128-byte lines of their rows: each XCD
    // takes a contiguous range of tiles
    if (!split_args(a, blk, nb, tab, st, ns)) blk = xcd_block(blk, nb);
    const int tid = threadIdx.x;
    const int M = a.nx / 2, R = a.ny / Q;
    const int ntx = (M + TX - 1) >> LG, s = (int)blk / ntx, kx0 = ((int)blk - s * ntx) << LG;
    // distance of consecutive q, Q of them per z (every offset inside the
    // spectrum fits 32 bits at the compiled lengths)
    const unsigned rq = (unsigned)a.gs;
    C2<T>* base = a.spec + (unsigned)(s * M + kx0);
    auto io = [](int u) { return (u >> LG) * ES + (u & (TX - 1)); };
    auto z0 = [](int u) { const int j = u / LT; return j * ES + (u - j * LT); };
    auto z1 = [](int u) { const int k0 = u / LT; return k0 * D1 * ES + (u - k0 * LT); };
    C2<T> v0[nunits<Io, NT>()][Q], v1[nunits<Z0, NT>()][D0], v2[nunits<Z1, NT>()][D1];
#pragma unroll
    for (int i = 0; i < nunits<Io, NT>(); ++i) {
        const int u = tid + i * NT, c = u & (TX - 1), z = u >> LG;
        const unsigned off = (unsigned)(z * Q) * rq + c;
#pragma unroll
        for (int q = 0; q < Q; ++q) v0[i][q] = C2<T>{T(0), T(0)};
        if (u < Io::N && kx0 + c < M) {
#pragma unroll
            for (int q = 0; q < Q; ++q) v0[i][q] = ldg(base + q * rq, off);
        }
    }
    for (int j = tid; j < NZ; j += NT) {
        wz[j] = ldg(a.wz, j);
        sz2[j] = ldg(a.sz2, j);
    }
#pragma unroll
    for (int i = 0; i < nunits<Io, NT>(); ++i) DFT<T, Q, false>::run(v0[i]);
    exchange_stages<HALF, NT, Io, Z0>(sm, v0, v1, tid, io, z0);
#pragma unroll
    for (int i = 0; i < nunits<Z0, NT>(); ++i) DFT<T, D0, false>::run(v1[i]);
    exchange_stages<HALF, NT, Z0, Z1>(sm, v1, v2, tid, z0, z1);
    // second z digit, divide by lambda N, second z digit back; the twiddles
    // W_nz^{k0 j} between the digits serve both directions
#pragma unroll
    for (int i = 0; i < nunits<Z1, NT>(); ++i) {
        const int u = tid + i * NT;
        if (u < Z1::N) {
            const int k0 = u / LT, o = u - k0 * LT;
            const double ly = ldg(a.sy2, s + R * (o >> LG)), lx = ldg(a.sx2, min(kx0 + (o & (TX - 1)), M - 1));
#pragma unroll
            for (int r = 1; r < D1; ++r) v2[i][r] = cmul(v2[i][r], wz[k0 * r]);
            DFT<T, D1, false>::run(v2[i]);
#pragma unroll
            for (int r = 0; r < D1; ++r) {
                const double lam = (sz2[k0 + D0 * r] + ly) + lx;   // -lambda
                const T f = lam == 0.0 ? T(0) : T(-a.inv_ntot * recip(lam));
                v2[i][r] = cscale(v2[i][r], f);
            }
            DFT<T, D1, true>::run(v2[i]);
#pragma unroll
            for (int r = 1; r < D1; ++r) v2[i][r] = cmulc(v2[i][r], wz[k0 * r]);
        }
    }
    // (arrays of their own: lanes without a unit would keep the old values alive)
    C2<T> w1[nunits<Z0, NT>()][D0], w0[nunits<Io, NT>()][Q];
    exchange_stages<HALF, NT, Z1, Z0>(sm, v2, w1, tid, z1, z0);
#pragma unroll
    for (int i = 0; i < nunits<Z0, NT>(); ++i) DFT<T, D0, true>::run(w1[i]);
    exchange_stages<HALF, NT, Z0, Io>(sm, w1, w0, tid, z0, io);
#pragma unroll
    for (int i = 0; i < nunits<Io, NT>(); ++i) {
        const int u = tid + i * NT, c = u & (TX - 1), z = u >> LG;
        const unsigned off = (unsigned)(z * Q) * rq + c;
        if (u < Io::N && kx0 + c < M) {
            DFT<T, Q, true>::run(w0[i]);
#pragma unroll
            for (int q = 0; q < Q; ++q) stg(base + q * rq, off, w0[i][q]);
        }
    }
}

}  // namespace
}  // namespace dnslab
