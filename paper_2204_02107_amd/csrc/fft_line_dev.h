// Kernels of the axis-by-axis FFT solve (fft_line.h), as templates that the
// fft_line_part.hip parts instantiate.  Tiles live in registers and are
// exchanged through LDS between digits as in fft_split_dev.h; the first digit
// of a transform is loaded from global memory, and the last one of a column
// transform is stored there, so a column pass of two digits has one exchange.
// Frequencies along the columns stay in digit order in memory: the inverse
// undoes it, and only the symbol has to know.
#pragma once

#include "fft_line.h"
#include "fft_split_dev.h"

namespace dnslab {
namespace {

template <typename T>
__device__ __forceinline__ bool line_args(LineArgs<T>& a, unsigned& blk, unsigned& nb, const BRec<LineArgs<T>>* tab,
                                          const unsigned* st, int ns) {
    blk = blockIdx.x;
    nb = gridDim.x;
    if (!tab) return false;
    const int e = batch_slot(st, ns);
    blk -= st[e];
    nb = tab[e].g[0];
    a = tab[e].a;
    return true;
}

// The W_n table: a copy in LDS, or global memory through the caches.
template <bool LDS, typename T>
struct WTab {
    C2<T>* lds;
    const C2<T>* g;
    __device__ __forceinline__ void stage(int n, int tid, int nt) const {
        if (LDS)
            for (int j = tid; j < n; j += nt) lds[j] = ldg(g, j);
    }
    __device__ __forceinline__ C2<T> operator[](int i) const { return LDS ? lds[i] : ldg(g, i); }
};

// Stages of an N-point transform of NL_ lines of a tile.
template <int N, int NL_, int NT_, int PAD>
struct LG {
    static constexpr SplitDigits dg = line_digits(N);
    static constexpr int NL = NL_, NT = NT_, ES = NL_;
    static constexpr int D0 = dg.d[0], D1 = dg.d[1], D2 = dg.d[2];
    static constexpr int S0 = N / D0, S1 = S0 / D1;
    using F0 = Stage<NL * (N / D0), D0, S0 * ES + PAD>;
    using F1 = Stage<NL * (N / D1), D1, S1 * ES>;
    using F2 = Stage<NL * (N / D2), D2, ES>;
    template <int S, int L>
    static __device__ __forceinline__ int place(int u) {   // first place of unit u
        const int t = u / NL;
        return (t / S) * L + t % S;
    }
    template <int S, int L>
    static __device__ __forceinline__ int digit(int u) {
        const int p = place<S, L>(u);
        return p * ES + p / S0 * PAD + u % NL;
    }
    static __device__ __forceinline__ int f0(int u) { return digit<S0, N>(u); }
    static __device__ __forceinline__ int f1(int u) { return digit<S1, S0>(u); }
    static __device__ __forceinline__ int f2(int u) { return digit<1, S1>(u); }
    static __device__ __forceinline__ int freq(int k) {
        const int k0 = k % D0, h = k / D0, k1 = h % D1, k2 = h / D1;
        return (k0 * S0 + k1 * S1 + k2) * ES + k0 * PAD;
    }
    // frequency at place p
    static __device__ __forceinline__ int at(int p) {
        const int k0 = p / S0, q = p - k0 * S0, k1 = q / S1;
        return k0 + D0 * (k1 + D1 * (q - k1 * S1));
    }
};

// x passes: NL lines per block; the pairs (k, m - k) as in the split passes,
// without a y digit.
template <class X, int M>
struct LineItem {
    int l, k, kb;
    unsigned pa, pb;
    bool in, on, two;
    __device__ __forceinline__ LineItem(int it, int blk, int nlines, int rs) {
        constexpr int H = (M + 1) / 2;
        l = it / H;
        k = it - l * H;
        kb = k ? M - k : M / 2;
        two = M % 2 == 0 || k != 0;
        const int line = blk * X::NL + l;
        in = it < X::NL * H;
        on = in && line < nlines;
        pa = (unsigned)line * (unsigned)rs + (unsigned)k;
        pb = (unsigned)line * (unsigned)rs + (unsigned)kb;
    }
};

template <typename T, int M>
__global__ __launch_bounds__(line_x_geom(M, (int)sizeof(T)).nt) void k_line_x_fwd(LineArgs<T> a,
                                                                                  const BRec<LineArgs<T>>* tab,
                                                                                  const unsigned* st, int ns) {
    constexpr LineGeom gm = line_x_geom(M, (int)sizeof(T));
    constexpr int NT = gm.nt, NI = (gm.nl * ((M + 1) / 2) + NT - 1) / NT;
    constexpr bool HALF = gm.half != 0;
    using X = LG<M, gm.nl, NT, gm.pad>;
    extern __shared__ unsigned char smem_raw[];
    C2<T>* s = reinterpret_cast<C2<T>*>(smem_raw);
    unsigned blk, nb;
    line_args(a, blk, nb, tab, st, ns);
    const int tid = threadIdx.x;
    const WTab<gm.wlds != 0, T> W{reinterpret_cast<C2<T>*>(smem_raw + gm.tile), a.wx};
    C2<T> v1[nunits<typename X::F0, NT>()][X::D0], v2[nunits<typename X::F1, NT>()][X::D1];
    const C2<T>* src = reinterpret_cast<const C2<T>*>(a.r);
#pragma unroll
    for (int i = 0; i < nunits<typename X::F0, NT>(); ++i) {
        const int u = tid + i * NT, l = u % X::NL, line = (int)blk * X::NL + l;
        const unsigned o = (unsigned)line * M + (unsigned)(u / X::NL);
#pragma unroll
        for (int r = 0; r < X::D0; ++r) v1[i][r] = C2<T>{T(0), T(0)};
        if (u < X::F0::N && line < a.nlines) {
#pragma unroll
            for (int r = 0; r < X::D0; ++r) v1[i][r] = ldg(src + r * X::S0, o);
        }
    }
    W.stage(M, tid, NT);
    if (gm.wlds) lds_barrier();
    x_digit<X, M, X::S0, false>(v1, W, tid);
    exchange_stages<HALF, NT, typename X::F0, typename X::F1>(s, v1, v2, tid, X::f0, X::f1);
    x_digit<X, M, X::S1, false>(v2, W, tid);
    C2<T> za[NI], zb[NI];
    auto gets = [&](auto p) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const LineItem<X, M> q(tid + i * NT, (int)blk, a.nlines, a.rs);
            if (q.in) {
                get<decltype(p)::value>(s, X::freq(q.k) + q.l, za[i]);
                if (q.two) get<decltype(p)::value>(s, X::freq(q.kb) + q.l, zb[i]);
            }
        }
    };
    if constexpr (X::dg.n == 3) {
        C2<T> v3[nunits<typename X::F2, NT>()][X::D2];
        exchange_stages<HALF, NT, typename X::F1, typename X::F2>(s, v2, v3, tid, X::f1, X::f2);
        x_digit<X, M, 1, false>(v3, W, tid);
        exchange<HALF>([&](auto p) { put_stage<typename X::F2, NT, decltype(p)::value>(s, v3, tid, X::f2); }, gets);
    } else {
        exchange<HALF>([&](auto p) { put_stage<typename X::F1, NT, decltype(p)::value>(s, v2, tid, X::f1); }, gets);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const LineItem<X, M> q(tid + i * NT, (int)blk, a.nlines, a.rs);
        if (!q.on) continue;
        const C2<T> w = ldg(a.tw, q.k), wm = C2<T>{-w.x, w.y};
        stg(a.spec, q.pa, q.k ? r2c_post(za[i], zb[i], w) : za[i]);
        if (q.two) stg(a.spec, q.pb, q.k ? r2c_post(zb[i], za[i], wm) : conj_(zb[i]));
    }
}

template <typename T, int M>
__global__ __launch_bounds__(line_x_geom(M, (int)sizeof(T)).nt) void k_line_x_inv(LineArgs<T> a,
                                                                                  const BRec<LineArgs<T>>* tab,
                                                                                  const unsigned* st, int ns) {
    constexpr LineGeom gm = line_x_geom(M, (int)sizeof(T));
    constexpr int NT = gm.nt, NI = (gm.nl * ((M + 1) / 2) + NT - 1) / NT;
    constexpr bool HALF = gm.half != 0;
    using X = LG<M, gm.nl, NT, gm.pad>;
    extern __shared__ unsigned char smem_raw[];
    C2<T>* s = reinterpret_cast<C2<T>*>(smem_raw);
    unsigned blk, nb;
    line_args(a, blk, nb, tab, st, ns);
    const int tid = threadIdx.x;
    const WTab<gm.wlds != 0, T> W{reinterpret_cast<C2<T>*>(smem_raw + gm.tile), a.wx};
    C2<T> xa[NI], xb[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const LineItem<X, M> q(tid + i * NT, (int)blk, a.nlines, a.rs);
        xa[i] = xb[i] = C2<T>{T(0), T(0)};
        if (q.on) {
            xa[i] = ldg(a.spec, q.pa);
            if (q.two) xb[i] = ldg(a.spec, q.pb);
        }
    }
    W.stage(M, tid, NT);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const LineItem<X, M> q(tid + i * NT, (int)blk, a.nlines, a.rs);
        if (!q.on) continue;
        const C2<T> w = ldg(a.tw, q.k), wm = C2<T>{-w.x, w.y};
        const C2<T> x = xa[i], y = xb[i];
        xa[i] = q.k ? c2r_pre(x, y, w) : cadd(x, x);
        xb[i] = q.k ? c2r_pre(y, x, wm) : conj_(cadd(y, y));
    }
    auto puts = [&](auto p) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const LineItem<X, M> q(tid + i * NT, (int)blk, a.nlines, a.rs);
            if (q.in) {
                put<decltype(p)::value>(s, X::freq(q.k) + q.l, xa[i]);
                if (q.two) put<decltype(p)::value>(s, X::freq(q.kb) + q.l, xb[i]);
            }
        }
    };
    C2<T> v1[nunits<typename X::F0, NT>()][X::D0], v2[nunits<typename X::F1, NT>()][X::D1];
    if constexpr (X::dg.n == 3) {
        C2<T> v3[nunits<typename X::F2, NT>()][X::D2];
        exchange<HALF>(puts, [&](auto p) { get_stage<typename X::F2, NT, decltype(p)::value>(s, v3, tid, X::f2); });
        x_digit<X, M, 1, true>(v3, W, tid);
        exchange_stages<HALF, NT, typename X::F2, typename X::F1>(s, v3, v2, tid, X::f2, X::f1);
    } else {
        exchange<HALF>(puts, [&](auto p) { get_stage<typename X::F1, NT, decltype(p)::value>(s, v2, tid, X::f1); });
    }
    x_digit<X, M, X::S1, true>(v2, W, tid);
    exchange_stages<HALF, NT, typename X::F1, typename X::F0>(s, v2, v1, tid, X::f1, X::f0);
    x_digit<X, M, X::S0, true>(v1, W, tid);
    C2<T>* dst = reinterpret_cast<C2<T>*>(a.p);
#pragma unroll
    for (int i = 0; i < nunits<typename X::F0, NT>(); ++i) {
        const int u = tid + i * NT, l = u % X::NL, line = (int)blk * X::NL + l;
        const unsigned o = (unsigned)line * M + (unsigned)(u / X::NL);
        if (u < X::F0::N && line < a.nlines) {
            const unsigned long long need = a.need ? need_word(a.need, line) : ~0ull;
#pragma unroll
            for (int r = 0; r < X::D0; ++r)
                if (need >> ((unsigned)(2 * (u / X::NL + r * X::S0)) >> a.seg_lg) & 1u) stg(dst + r * X::S0, o, v1[i][r]);
        }
    }
}

// Column passes along N rows of TX consecutive kx.
template <typename T, int N, int MODE>
__global__ __launch_bounds__(line_c_geom(N, (int)sizeof(T)).nt) void k_line_cols(LineArgs<T> a,
                                                                                 const BRec<LineArgs<T>>* tab,
                                                                                 const unsigned* st, int ns) {
    constexpr LineGeom gm = line_c_geom(N, (int)sizeof(T));
    constexpr int NT = gm.nt, TX = gm.nl;
    constexpr bool HALF = gm.half != 0;
    using X = LG<N, TX, NT, gm.pad>;
    using F0 = typename X::F0;
    using FL = std::conditional_t<X::dg.n == 3, typename X::F2, typename X::F1>;   // the last digit
    constexpr int DL = FL::D;
    constexpr int U0 = nunits<F0, NT>(), UL = nunits<FL, NT>();
    extern __shared__ unsigned char smem_raw[];
    C2<T>* s = reinterpret_cast<C2<T>*>(smem_raw);
    unsigned blk, nb;
    if (!line_args(a, blk, nb, tab, st, ns)) blk = xcd_block(blk, nb);
    const int tid = threadIdx.x;
    const WTab<gm.wlds != 0, T> W{reinterpret_cast<C2<T>*>(smem_raw + gm.tile), a.wc};
    const int M = a.nx / 2, ntx = (M + TX - 1) / TX, plane = (int)blk / ntx, kx0 = ((int)blk - plane * ntx) * TX;
    C2<T>* base = a.spec + (size_t)plane * (size_t)a.pstr + kx0;
    const unsigned rstr = (unsigned)a.rstr;
    auto fl = [](int u) { return X::dg.n == 3 ? X::f2(u) : X::f1(u); };
    // last digit: unit u holds the consecutive places p0(u) ..
    auto p0 = [](int u) { return (u / TX) * DL; };
    C2<T> vl[UL][DL];
    // the middle digits: v0 -> vl (forward) through the second digit of three
    auto to_last = [&](C2<T> (&v0)[U0][X::D0]) {
        x_digit<X, N, X::S0, false>(v0, W, tid);
        if constexpr (X::dg.n == 3) {
            C2<T> v1[nunits<typename X::F1, NT>()][X::D1];
            exchange_stages<HALF, NT, F0, typename X::F1>(s, v0, v1, tid, X::f0, X::f1);
            x_digit<X, N, X::S1, false>(v1, W, tid);
            exchange_stages<HALF, NT, typename X::F1, FL>(s, v1, vl, tid, X::f1, fl);
        } else {
            exchange_stages<HALF, NT, F0, FL>(s, v0, vl, tid, X::f0, fl);
        }
        x_digit<X, N, 1, false>(vl, W, tid);
    };
    auto from_last = [&](C2<T> (&v0)[U0][X::D0]) {
        x_digit<X, N, 1, true>(vl, W, tid);
        if constexpr (X::dg.n == 3) {
            C2<T> v1[nunits<typename X::F1, NT>()][X::D1];
            exchange_stages<HALF, NT, FL, typename X::F1>(s, vl, v1, tid, fl, X::f1);
            x_digit<X, N, X::S1, true>(v1, W, tid);
            exchange_stages<HALF, NT, typename X::F1, F0>(s, v1, v0, tid, X::f1, X::f0);
        } else {
            exchange_stages<HALF, NT, FL, F0>(s, vl, v0, tid, fl, X::f0);
        }
        x_digit<X, N, X::S0, true>(v0, W, tid);
    };
    if constexpr (MODE == 1) {
#pragma unroll
        for (int i = 0; i < UL; ++i) {
            const int u = tid + i * NT, c = u % TX;
            const unsigned o = (unsigned)p0(u) * rstr + (unsigned)c;
#pragma unroll
            for (int r = 0; r < DL; ++r) vl[i][r] = C2<T>{T(0), T(0)};
            if (u < FL::N && kx0 + c < M) {
#pragma unroll
                for (int r = 0; r < DL; ++r) vl[i][r] = ldg(base + (unsigned)r * rstr, o);
            }
        }
    } else {
        C2<T> v0[U0][X::D0];
#pragma unroll
        for (int i = 0; i < U0; ++i) {
            const int u = tid + i * NT, c = u % TX;
            const unsigned o = (unsigned)(u / TX) * rstr + (unsigned)c;
#pragma unroll
            for (int r = 0; r < X::D0; ++r) v0[i][r] = C2<T>{T(0), T(0)};
            if (u < F0::N && kx0 + c < M) {
#pragma unroll
                for (int r = 0; r < X::D0; ++r) v0[i][r] = ldg(base + (unsigned)(r * X::S0) * rstr, o);
            }
        }
        W.stage(N, tid, NT);
        if (gm.wlds) lds_barrier();
        to_last(v0);
    }
    if constexpr (MODE == 0) {
#pragma unroll
        for (int i = 0; i < UL; ++i) {
            const int u = tid + i * NT, c = u % TX;
            const unsigned o = (unsigned)p0(u) * rstr + (unsigned)c;
            if (u < FL::N && kx0 + c < M) {
#pragma unroll
                for (int r = 0; r < DL; ++r) stg(base + (unsigned)r * rstr, o, vl[i][r]);
            }
        }
        return;
    }
    if constexpr (MODE == 1) {
        W.stage(N, tid, NT);
        if (gm.wlds) lds_barrier();
    }
    if constexpr (MODE == 2) {
        // the plane's frequency, from its place
        int kp = plane;
        if (a.np) {
            const int n = a.nplanes, s0 = n / a.d0, s1 = s0 / a.d1;
            const int k0 = plane / s0, q = plane - k0 * s0, k1 = q / s1;
            kp = k0 + a.d0 * (k1 + a.d1 * (q - k1 * s1));
        }
        const double lp = ldg(a.sp2, kp);
#pragma unroll
        for (int i = 0; i < UL; ++i) {
            const int u = tid + i * NT;
            if (u < FL::N) {
                const double lx = ldg(a.sx2, min(kx0 + u % TX, M - 1));
#pragma unroll
                for (int r = 0; r < DL; ++r) {
                    const double lam = (ldg(a.sc2, X::at(p0(u) + r)) + lp) + lx;   // -lambda
                    const T f = lam == 0.0 ? T(0) : T(-a.inv_ntot * recip(lam));
                    vl[i][r] = cscale(vl[i][r], f);
                }
            }
        }
    }
    C2<T> w0[U0][X::D0];
    from_last(w0);
#pragma unroll
    for (int i = 0; i < U0; ++i) {
        const int u = tid + i * NT, c = u % TX;
        const unsigned o = (unsigned)(u / TX) * rstr + (unsigned)c;
        if (u < F0::N && kx0 + c < M) {
#pragma unroll
            for (int r = 0; r < X::D0; ++r) stg(base + (unsigned)(r * X::S0) * rstr, o, w0[i][r]);
        }
    }
}

}  // namespace
}  // namespace dnslab
