// Device building blocks shared by the FFT kernels (fft.hip, fft_split.hip):
// complex arithmetic, in-register DFTs, the real-transform twist and the
// reciprocal of the spectral symbol.
#pragma once

#include "common.h"

namespace dnslab {
namespace {

template <typename T>
__device__ __forceinline__ C2<T> cadd(C2<T> a, C2<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__device__ __forceinline__ C2<T> csub(C2<T> a, C2<T> b) { return {a.x - b.x, a.y - b.y}; }
template <typename T>
__device__ __forceinline__ C2<T> cscale(C2<T> a, T s) { return {a.x * s, a.y * s}; }
template <typename T>
__device__ __forceinline__ C2<T> cmul(C2<T> a, C2<T> b) {
    return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
// a * conj(b)
template <typename T>
__device__ __forceinline__ C2<T> cmulc(C2<T> a, C2<T> b) {
    return {a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y};
}
template <typename T>
__device__ __forceinline__ C2<T> conj_(C2<T> a) { return {a.x, -a.y}; }
// multiply by -i (forward sign) or +i (inverse sign)
template <typename T, bool INV>
__device__ __forceinline__ C2<T> rot(C2<T> a) {
    return INV ? C2<T>{-a.y, a.x} : C2<T>{a.y, -a.x};
}

// In-register DFT of length R with kernel e^{-+2 pi i r m / R}.
template <typename T, int R, bool INV>
struct DFT;

template <typename T, bool INV>
struct DFT<T, 2, INV> {
    static __device__ __forceinline__ void run(C2<T>* v) {
        const C2<T> a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    }
};

template <typename T, bool INV>
struct DFT<T, 4, INV> {
    static __device__ __forceinline__ void run(C2<T>* v) {
        const C2<T> t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
        const C2<T> t2 = cadd(v[1], v[3]), t3 = rot<T, INV>(csub(v[1], v[3]));
        v[0] = cadd(t0, t2);
        v[2] = csub(t0, t2);
        v[1] = cadd(t1, t3);
        v[3] = csub(t1, t3);
    }
};

template <typename T, bool INV>
struct DFT<T, 8, INV> {
    static __device__ __forceinline__ void run(C2<T>* v) {
        C2<T> e[4] = {v[0], v[2], v[4], v[6]};
        C2<T> o[4] = {v[1], v[3], v[5], v[7]};
        DFT<T, 4, INV>::run(e);
        DFT<T, 4, INV>::run(o);
        const T h = T(0.70710678118654752440);
        // o[m] *= w8^m, w8 = e^{-+ i pi / 4}
        const C2<T> o1 = INV ? C2<T>{h * (o[1].x - o[1].y), h * (o[1].x + o[1].y)}
                             : C2<T>{h * (o[1].x + o[1].y), h * (o[1].y - o[1].x)};
        const C2<T> o2 = rot<T, INV>(o[2]);
        const C2<T> o3 = INV ? C2<T>{-h * (o[3].x + o[3].y), h * (o[3].x - o[3].y)}
                             : C2<T>{h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y)};
        v[0] = cadd(e[0], o[0]);
        v[4] = csub(e[0], o[0]);
        v[1] = cadd(e[1], o1);
        v[5] = csub(e[1], o1);
        v[2] = cadd(e[2], o2);
        v[6] = csub(e[2], o2);
        v[3] = cadd(e[3], o3);
        v[7] = csub(e[3], o3);
    }
};

template <typename T, bool INV>
struct DFT<T, 3, INV> {
    static __device__ __forceinline__ void run(C2<T>* v) {
        const T h = T(0.86602540378443864676);   // sqrt(3)/2
        const C2<T> t = cadd(v[1], v[2]);
        const C2<T> sd = rot<T, INV>(csub(v[1], v[2]));
        const C2<T> m = {v[0].x - T(0.5) * t.x, v[0].y - T(0.5) * t.y};
        v[0] = cadd(v[0], t);
        v[1] = {m.x + h * sd.x, m.y + h * sd.y};
        v[2] = {m.x - h * sd.x, m.y - h * sd.y};
    }
};

// cos(2 pi j / 288), j = 0..72, correctly rounded: every root of unity the
// in-register DFTs below need (orders 6, 9, 12, 16, 18 divide 288).
constexpr double COS288[73] = {
    1, 0.99976202707990913243, 0.99904822158185779823, 0.99785892323860347908, 0.9961946980917455452,
    0.99405633822231964647, 0.99144486137381038215, 0.9883615104677606622, 0.98480775301220802032,
    0.98078528040323043058, 0.97629600711993336226, 0.97134206981326143282, 0.96592582628906831221,
    0.96004985438592871372, 0.95371695074822693261, 0.94693012949510568799, 0.93969262078590842791,
    0.93200786928279855115, 0.92387953251128673848, 0.91531147911944710227, 0.90630778703664993667,
    0.89687274153268825572, 0.8870108331782217137, 0.87672675570750768781, 0.86602540378443859659,
    0.85491187067294660551, 0.84339144581288572056, 0.83146961230254523567, 0.81915204428899179856,
    0.80644460426748254545, 0.79335334029123516508, 0.77988448309288183058, 0.76604444311897801345,
    0.75183980747897738439, 0.73727733681012408429, 0.72236396205975561546, 0.70710678118654757274,
    0.69151305578226940352, 0.67559020761566024316, 0.65934581510006884386, 0.64278760968653936292,
    0.62592347218405908205, 0.60876142900872065589, 0.59130964836358235193, 0.5735764363510460484,
    0.55557023301960217765, 0.53729960834682388704, 0.51877325816052144436, 0.5, 0.48098876891938763256,
    0.4617486132350339112, 0.44228869021900130143, 0.42261826174069944129, 0.40274668985873723903,
    0.38268343236508978178, 0.36243803828370163567, 0.34202014332566871291, 0.32143946530316158672,
    0.3007057995042731191, 0.2798290140309920293, 0.25881904510252073948, 0.23768589232617309825,
    0.21643961393810287608, 0.19509032201612827584, 0.17364817766693035894, 0.15212338618991669281,
    0.13052619222005160116, 0.1088668748519645707, 0.087155742747658179748, 0.065403129230143061679,
    0.043619387365336000084, 0.021814885034561120464, 0.0
};
constexpr double cos288(int j) {
    j = j % 288;
    if (j > 144) j = 288 - j;
    return j <= 72 ? COS288[j] : -COS288[144 - j];
}

// a * W_N^K (forward, W = e^{-2 pi i / N}) or its conjugate (INV), K and N
// known at compile time; multiples of a quarter turn move components only.
template <typename T, int N, int K, bool INV>
__device__ __forceinline__ C2<T> cmul_root(C2<T> a) {
    static_assert(288 % N == 0, "root order");
    constexpr int j = (K % N) * (288 / N);
    if constexpr (j == 0) return a;
    else if constexpr (j == 72) return rot<T, INV>(a);
    else if constexpr (j == 144) return C2<T>{-a.x, -a.y};
    else if constexpr (j == 216) return rot<T, !INV>(a);
    else {
        constexpr T c = T(cos288(j)), s = T(cos288(j + 216));   // sin = cos(phi - pi/2)
        // forward: (x + i y)(c - i s)
        return INV ? C2<T>{a.x * c - a.y * s, a.x * s + a.y * c} : C2<T>{a.x * c + a.y * s, a.y * c - a.x * s};
    }
}

// v[A] *= W_N^{a b} for one b, by recursion over a (compile-time indices).
template <typename T, int N, int B_, int A_, int A0, bool INV>
__device__ __forceinline__ void twiddle_row(C2<T>* y) {
    if constexpr (A0 < A_) {
        y[A0] = cmul_root<T, N, A0 * B_, INV>(y[A0]);
        twiddle_row<T, N, B_, A_, A0 + 1, INV>(y);
    }
}
template <typename T, int A, int B, int B0, bool INV>
__device__ __forceinline__ void ct_inner(const C2<T>* v, C2<T> (*y)[A]) {
    if constexpr (B0 < B) {
#pragma unroll
        for (int a = 0; a < A; ++a) y[B0][a] = v[B * a + B0];
        DFT<T, A, INV>::run(y[B0]);
        if constexpr (B0 > 0) twiddle_row<T, A * B, B0, A, 1, INV>(y[B0]);
        ct_inner<T, A, B, B0 + 1, INV>(v, y);
    }
}
// Length A * B from lengths A and B: with n = B a + b, k = ka + A kb,
// X[k] = sum_b W_B^{b kb} W_{AB}^{b ka} sum_a x[n] W_A^{a ka}.
template <typename T, int A, int B, bool INV>
__device__ __forceinline__ void dft_ct(C2<T>* v) {
    C2<T> y[B][A];
    ct_inner<T, A, B, 0, INV>(v, y);
#pragma unroll
    for (int ka = 0; ka < A; ++ka) {
        C2<T> z[B];
#pragma unroll
        for (int b = 0; b < B; ++b) z[b] = y[b][ka];
        DFT<T, B, INV>::run(z);
#pragma unroll
        for (int kb = 0; kb < B; ++kb) v[ka + A * kb] = z[kb];
    }
}
template <typename T, bool INV>
struct DFT<T, 6, INV> {
    static __device__ __forceinline__ void run(C2<T>* v) { dft_ct<T, 3, 2, INV>(v); }
};
template <typename T, bool INV>
struct DFT<T, 9, INV> {
    static __device__ __forceinline__ void run(C2<T>* v) { dft_ct<T, 3, 3, INV>(v); }
};
template <typename T, bool INV>
struct DFT<T, 12, INV> {
    static __device__ __forceinline__ void run(C2<T>* v) { dft_ct<T, 4, 3, INV>(v); }
};
template <typename T, bool INV>
struct DFT<T, 16, INV> {
    static __device__ __forceinline__ void run(C2<T>* v) { dft_ct<T, 4, 4, INV>(v); }
};
template <typename T, bool INV>
struct DFT<T, 18, INV> {
    static __device__ __forceinline__ void run(C2<T>* v) { dft_ct<T, 6, 3, INV>(v); }
};

// X[k] of the real transform from Z = FFT(x_even + i x_odd):
// E = (Z[k] + conj Z[m-k])/2, O = -i (Z[k] - conj Z[m-k])/2, X[k] = E + w^k O.
template <typename T>
__device__ __forceinline__ C2<T> r2c_post(C2<T> za, C2<T> zb, C2<T> w) {
    const C2<T> zc = conj_(zb);
    const C2<T> e = cscale(cadd(za, zc), T(0.5));
    const C2<T> o = cscale(rot<T, false>(csub(za, zc)), T(0.5));
    return cadd(e, cmul(w, o));
}
// Z[k] for the inverse from X[k], X[m-k] (unnormalised: twice the even/odd
// spectra): E = X[k] + conj X[m-k], O = (X[k] - conj X[m-k]) conj(w^k), Z = E + i O.
template <typename T>
__device__ __forceinline__ C2<T> c2r_pre(C2<T> xa, C2<T> xb, C2<T> w) {
    const C2<T> xc = conj_(xb);
    const C2<T> e = cadd(xa, xc);
    const C2<T> o = cmulc(csub(xa, xc), w);
    return cadd(e, rot<T, true>(o));
}

// 1/x to about one ulp: hardware reciprocal refined by two Newton steps.
__device__ __forceinline__ double recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    r = fma(r, fma(-x, r, 1.0), r);
    return r;
}

}  // namespace
}  // namespace dnslab
