// Complex arithmetic and small DFTs of the Stockham FFT passes for gfx950
// (fft_col.hpp: column tiles; fft_row.hpp: rows of the x passes).
//
// Stage with span NS (product of the radices already applied), butterfly j:
//   k = j mod NS
//   v[r] = x[j + r L/R] * W_{NS R}^{r k}
//   v = DFT_R(v)
//   x'[(j div NS) NS R + k + r NS] = v[r]
// One stage of radix R0, then radix-8 stages: lengths R0 8^k with R0 = 2, 4, 8,
// 16, 3, 6, 12, 5, 10 or 20 (first_radix, col_radix), that is 2^m, 3 2^m and
// 5 2^m.  The forward transform uses e^{-2 pi i/L}; the inverse
// uses e^{+2 pi i/L} and is unnormalised.  Twiddles come from a table
// tw[m] = e^{-2 pi i m/L}, m < L, built on the host in double precision.
#pragma once
#include <hip/hip_runtime.h>

namespace llgx {

template <typename T> struct cplx;
template <> struct cplx<float> { using type = float2; };
template <> struct cplx<double> { using type = double2; };
template <typename T> using cx = typename cplx<T>::type;

template <typename C> __device__ __forceinline__ C cadd(C a, C b) { return C{a.x + b.x, a.y + b.y}; }
template <typename C> __device__ __forceinline__ C csub(C a, C b) { return C{a.x - b.x, a.y - b.y}; }
template <typename C> __device__ __forceinline__ C cmul(C a, C b) {
    return C{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
// a * conj(b)
template <typename C> __device__ __forceinline__ C cmulc(C a, C b) {
    return C{a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y};
}
template <typename C> __device__ __forceinline__ C cconj(C a) { return C{a.x, -a.y}; }
// multiply by -i (forward) or +i (inverse)
template <bool INV, typename C> __device__ __forceinline__ C rot90(C a) {
    return INV ? C{-a.y, a.x} : C{a.y, -a.x};
}

template <bool INV, typename C> __device__ __forceinline__ void dft2(C& a0, C& a1) {
    C t = a0;
    a0 = cadd(t, a1);
    a1 = csub(t, a1);
}

template <bool INV, typename C> __device__ __forceinline__ void dft4(C& a0, C& a1, C& a2, C& a3) {
    C t0 = cadd(a0, a2), t1 = csub(a0, a2);
    C t2 = cadd(a1, a3), t3 = rot90<INV>(csub(a1, a3));
    a0 = cadd(t0, t2);
    a2 = csub(t0, t2);
    a1 = cadd(t1, t3);
    a3 = csub(t1, t3);
}

template <bool INV, typename C> __device__ __forceinline__ void dft8(C* v) {
    using T = decltype(v[0].x);
    const T s = T(0.70710678118654752440084436210484903928);
    C e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
    C o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
    dft4<INV>(e0, e1, e2, e3);
    dft4<INV>(o0, o1, o2, o3);
    // o_k *= W8^k, W8 = e^{-+ 2 pi i / 8}
    C w1 = INV ? C{s * (o1.x - o1.y), s * (o1.x + o1.y)} : C{s * (o1.x + o1.y), s * (o1.y - o1.x)};
    C w2 = rot90<INV>(o2);
    C w3 = INV ? C{-s * (o3.x + o3.y), s * (o3.x - o3.y)} : C{s * (o3.y - o3.x), -s * (o3.x + o3.y)};
    v[0] = cadd(e0, o0);
    v[4] = csub(e0, o0);
    v[1] = cadd(e1, w1);
    v[5] = csub(e1, w1);
    v[2] = cadd(e2, w2);
    v[6] = csub(e2, w2);
    v[3] = cadd(e3, w3);
    v[7] = csub(e3, w3);
}

template <bool INV, typename C> __device__ __forceinline__ void dft3(C* v) {
    using T = decltype(v[0].x);
    const T h = T(0.5), s = T(0.86602540378443864676372317075293618347);  // sin(2 pi / 3)
    const C t = cadd(v[1], v[2]);
    const C d = rot90<INV>(csub(v[1], v[2]));
    const C m = C{v[0].x - h * t.x, v[0].y - h * t.y};
    v[0] = cadd(v[0], t);
    v[1] = C{m.x + s * d.x, m.y + s * d.y};
    v[2] = C{m.x - s * d.x, m.y - s * d.y};
}

template <bool INV, typename C> __device__ __forceinline__ void dft5(C* v) {
    using T = decltype(v[0].x);
    // cos and sin of 2 pi / 5 and 4 pi / 5
    const T c1 = T(0.30901699437494742410229341718281905886), c2 = T(-0.80901699437494742410229341718281905886);
    const T s1 = T(0.95105651629515357211643933337938214340), s2 = T(0.58778525229247312916870595463907276860);
    const C p = cadd(v[1], v[4]), q = cadd(v[2], v[3]);
    const C d = csub(v[1], v[4]), e = csub(v[2], v[3]);
    const C a{v[0].x + (c1 * p.x + c2 * q.x), v[0].y + (c1 * p.y + c2 * q.y)};
    const C b{v[0].x + (c2 * p.x + c1 * q.x), v[0].y + (c2 * p.y + c1 * q.y)};
    const C f = rot90<INV>(C{s1 * d.x + s2 * e.x, s1 * d.y + s2 * e.y});
    const C g = rot90<INV>(C{s2 * d.x - s1 * e.x, s2 * d.y - s1 * e.y});
    v[0] = cadd(v[0], cadd(p, q));
    v[1] = cadd(a, f);
    v[4] = csub(a, f);
    v[2] = cadd(b, g);
    v[3] = csub(b, g);
}

template <bool INV, typename C> __device__ __forceinline__ void dft16(C* v) {
    using T = decltype(v[0].x);
    const T s = T(0.70710678118654752440084436210484903928);
    const T c1 = T(0.92387953251128675612818318939678828682), s1 = T(0.38268343236508977172845998403039886676);
    C e[8], o[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        e[i] = v[2 * i];
        o[i] = v[2 * i + 1];
    }
    dft8<INV>(e);
    dft8<INV>(o);
    const T wx[8] = {T(1), c1, s, s1, T(0), -s1, -s, -c1};
    const T wy[8] = {T(0), -s1, -s, -c1, T(-1), -c1, -s, -s1};
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const C w{wx[k], wy[k]};
        const C t = k == 0 ? o[0] : k == 4 ? rot90<INV>(o[4]) : INV ? cmulc(o[k], w) : cmul(o[k], w);
        v[k] = cadd(e[k], t);
        v[k + 8] = csub(e[k], t);
    }
}

template <int R, bool INV, typename C> __device__ __forceinline__ void dft_r(C* v);

// R = A B with A, B coprime, without twiddles (Good and Thomas): input
// n = (B n1 + A n2) mod R, output k with k = k1 mod A, k = k2 mod B
template <int A, int B, bool INV, typename C> __device__ __forceinline__ void dft_coprime(C* v) {
    constexpr int R = A * B;
    C x[B][A];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
#pragma unroll
        for (int n1 = 0; n1 < A; ++n1) x[n2][n1] = v[(B * n1 + A * n2) % R];
        dft_r<A, INV>(x[n2]);
    }
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
        C y[B];
#pragma unroll
        for (int n2 = 0; n2 < B; ++n2) y[n2] = x[n2][k1];
        dft_r<B, INV>(y);
#pragma unroll
        for (int k = k1; k < R; k += A) v[k] = y[k % B];
    }
}

template <int R, bool INV, typename C> __device__ __forceinline__ void dft_r(C* v) {
    if constexpr (R == 2) {
        dft2<INV>(v[0], v[1]);
    } else if constexpr (R == 4) {
        dft4<INV>(v[0], v[1], v[2], v[3]);
    } else if constexpr (R == 8) {
        dft8<INV>(v);
    } else if constexpr (R == 16) {
        dft16<INV>(v);
    } else if constexpr (R == 3) {
        dft3<INV>(v);
    } else if constexpr (R == 5) {
        dft5<INV>(v);
    } else if constexpr (R == 6) {
        dft_coprime<2, 3, INV>(v);
    } else if constexpr (R == 10) {
        dft_coprime<2, 5, INV>(v);
    } else if constexpr (R == 12) {
        dft_coprime<4, 3, INV>(v);
    } else {
        static_assert(R == 20, "radix");
        dft_coprime<4, 5, INV>(v);
    }
}

constexpr int ilog2(int n) { return n <= 1 ? 0 : 1 + ilog2(n / 2); }

// radix of the first stage: L = first_radix(L) 8^k
constexpr int first_radix(int L) {
    const int odd = L % 3 == 0 ? 3 : L % 5 == 0 ? 5 : 1;
    const int m = ilog2(L / odd) % 3;
    return m == 1 ? 2 * odd : m == 2 ? 4 * odd : odd == 1 ? 8 : odd;
}
constexpr int fft_stages(int L, int R0) { return 1 + ilog2(L / R0) / 3; }

// The lengths the passes are built for: powers of two and, for spectra stored
// in the working precision, 3 2^m and 5 2^m from 24 on (those that hold a whole
// radix-8 stage).  An axis of n cells is padded to the smallest that is at least
// 2n - 1 (pad_length in llgx_api.hip).  The x passes transform half-length
// rows, LX = Px/2 from the same list.
#define LLGX_POW2_LENGTHS(M) M(2) M(4) M(8) M(16) M(32) M(64) M(128) M(256) M(512) M(1024)
#define LLGX_POW2_LENGTHS_LONG(M) M(2048)
#define LLGX_MIXED_LENGTHS(M) M(24) M(40) M(48) M(80) M(96) M(160) M(192) M(320) M(384) M(640) M(768)
#define LLGX_MIXED_LENGTHS_LONG(M) M(1280) M(1536)
#if LLGX_INST == 1 || LLGX_INST == 2  // 16-bit spectra
#define LLGX_FFT_LENGTHS(M) LLGX_POW2_LENGTHS(M)
#define LLGX_FFT_LENGTHS_LONG(M) LLGX_POW2_LENGTHS_LONG(M)
#else
#define LLGX_FFT_LENGTHS(M) LLGX_POW2_LENGTHS(M) LLGX_MIXED_LENGTHS(M)
#define LLGX_FFT_LENGTHS_LONG(M) LLGX_POW2_LENGTHS_LONG(M) LLGX_MIXED_LENGTHS_LONG(M)
#endif

}  // namespace llgx
