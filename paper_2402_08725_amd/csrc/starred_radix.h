// Complex helpers and short DFTs held in registers, for the FFT kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace starred {

__device__ __forceinline__ float2 cmul(float2 a, float2 b)
{
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cmulc(float2 a, float2 b)  // a * conj(b)
{
    return make_float2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
__device__ __forceinline__ float2 conjf2(float2 a) { return make_float2(a.x, -a.y); }
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }

// v <- the R-point DFT of v in place, sign -1 (forward) or +1 (INV). R = 2, 3, 4, 5 directly;
// 8, 9 and 16 as A x B with the twiddles W_R^(n2 k1) between the two; products of coprime
// factors (6, 10, 12, 15) by the prime-factor index map, which needs no twiddles.
template <int R, bool INV>
__device__ __forceinline__ void dft(float2 (&v)[R]);

template <bool INV>
__device__ __forceinline__ void dft2(float2 (&v)[2])
{
    const float2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
}

template <bool INV>
__device__ __forceinline__ void dft3(float2 (&v)[3])
{
    const float s1 = INV ? 0.86602540378443865f : -0.86602540378443865f;
    const float2 a = v[0], t = cadd(v[1], v[2]), d = csub(v[1], v[2]);
    const float2 m = make_float2(a.x - 0.5f * t.x, a.y - 0.5f * t.y);
    const float2 id = make_float2(-s1 * d.y, s1 * d.x);
    v[0] = cadd(a, t);
    v[1] = cadd(m, id);
    v[2] = csub(m, id);
}

template <bool INV>
__device__ __forceinline__ void dft4(float2 (&v)[4])
{
    const float2 a0 = cadd(v[0], v[2]), a1 = csub(v[0], v[2]);
    const float2 b0 = cadd(v[1], v[3]), b1 = csub(v[1], v[3]);
    const float2 rb = INV ? make_float2(-b1.y, b1.x) : make_float2(b1.y, -b1.x);
    v[0] = cadd(a0, b0);
    v[2] = csub(a0, b0);
    v[1] = cadd(a1, rb);
    v[3] = csub(a1, rb);
}

template <bool INV>
__device__ __forceinline__ void dft5(float2 (&v)[5])
{
    const float c1 = 0.30901699437494742f, c2 = -0.80901699437494742f;
    const float sg = INV ? 1.f : -1.f;
    const float s1 = sg * 0.95105651629515357f, s2 = sg * 0.58778525229247313f;
    const float2 a = v[0];
    const float2 t1 = cadd(v[1], v[4]), d1 = csub(v[1], v[4]);
    const float2 t2 = cadd(v[2], v[3]), d2 = csub(v[2], v[3]);
    const float2 m1 = make_float2(a.x + c1 * t1.x + c2 * t2.x, a.y + c1 * t1.y + c2 * t2.y);
    const float2 m2 = make_float2(a.x + c2 * t1.x + c1 * t2.x, a.y + c2 * t1.y + c1 * t2.y);
    const float2 u1 = make_float2(-(s1 * d1.y + s2 * d2.y), s1 * d1.x + s2 * d2.x);
    const float2 u2 = make_float2(-(s2 * d1.y - s1 * d2.y), s2 * d1.x - s1 * d2.x);
    v[0] = cadd(a, cadd(t1, t2));
    v[1] = cadd(m1, u1);
    v[4] = csub(m1, u1);
    v[2] = cadd(m2, u2);
    v[3] = csub(m2, u2);
}

// e^{-2 pi i m / R} for the composite lengths that need twiddles
template <int R>
struct RadixTw;
template <>
struct RadixTw<8> {
    static constexpr float c[8] = {1.f, 0.70710678118654752f, 0.f, -0.70710678118654752f};
    static constexpr float s[8] = {0.f, 0.70710678118654752f, 1.f, 0.70710678118654752f};
};
template <>
struct RadixTw<9> {
    static constexpr float c[9] = {1.f, 0.76604444311897804f, 0.17364817766693035f, -0.5f, -0.93969262078590838f};
    static constexpr float s[9] = {0.f, 0.64278760968653933f, 0.98480775301220806f, 0.86602540378443865f,
                                   0.34202014332566873f};
};
template <>
struct RadixTw<16> {
    static constexpr float c[16] = {1.f, 0.92387953251128674f, 0.70710678118654752f, 0.38268343236508977f, 0.f,
                                    -0.38268343236508977f, -0.70710678118654752f, -0.92387953251128674f, -1.f,
                                    -0.92387953251128674f};
    static constexpr float s[16] = {0.f, 0.38268343236508977f, 0.70710678118654752f, 0.92387953251128674f, 1.f,
                                    0.92387953251128674f, 0.70710678118654752f, 0.38268343236508977f, 0.f,
                                    -0.38268343236508977f};
};

template <int R, bool INV>
__device__ __forceinline__ float2 radix_twiddle(float2 v, int m)
{
    if (m == 0) return v;
    if (4 * m == R) return INV ? make_float2(-v.y, v.x) : make_float2(v.y, -v.x);
    const float c = RadixTw<R>::c[m], s = RadixTw<R>::s[m];  // W = c - i s (forward), c + i s (inverse)
    return INV ? make_float2(v.x * c - v.y * s, v.y * c + v.x * s) : make_float2(v.x * c + v.y * s, v.y * c - v.x * s);
}

// n = B n1 + n2, k = k1 + A k2
template <int A, int B, bool INV>
__device__ __forceinline__ void dft_ct(float2 (&v)[A * B])
{
    float2 y[A][B];
    #pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
        float2 u[A];
        #pragma unroll
        for (int n1 = 0; n1 < A; ++n1) u[n1] = v[B * n1 + n2];
        dft<A, INV>(u);
        #pragma unroll
        for (int k1 = 0; k1 < A; ++k1) y[k1][n2] = radix_twiddle<A * B, INV>(u[k1], n2 * k1);
    }
    #pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
        dft<B, INV>(y[k1]);
        #pragma unroll
        for (int k2 = 0; k2 < B; ++k2) v[k1 + A * k2] = y[k1][k2];
    }
}

// coprime A, B: n = (B n1 + A n2) mod AB, k1 = k mod A, k2 = k mod B
template <int A, int B, bool INV>
__device__ __forceinline__ void dft_pf(float2 (&v)[A * B])
{
    float2 y[A][B];
    #pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
        float2 u[A];
        #pragma unroll
        for (int n1 = 0; n1 < A; ++n1) u[n1] = v[(B * n1 + A * n2) % (A * B)];
        dft<A, INV>(u);
        #pragma unroll
        for (int k1 = 0; k1 < A; ++k1) y[k1][n2] = u[k1];
    }
    #pragma unroll
    for (int k1 = 0; k1 < A; ++k1) dft<B, INV>(y[k1]);
    #pragma unroll
    for (int k = 0; k < A * B; ++k) v[k] = y[k % A][k % B];
}

template <int R, bool INV>
__device__ __forceinline__ void dft(float2 (&v)[R])
{
    static_assert((R >= 2 && R <= 6) || R == 8 || R == 9 || R == 10 || R == 12 || R == 15 || R == 16, "radix");
    if constexpr (R == 2) dft2<INV>(v);
    else if constexpr (R == 3) dft3<INV>(v);
    else if constexpr (R == 4) dft4<INV>(v);
    else if constexpr (R == 5) dft5<INV>(v);
    else if constexpr (R == 6) dft_pf<2, 3, INV>(v);
    else if constexpr (R == 8) dft_ct<2, 4, INV>(v);
    else if constexpr (R == 9) dft_ct<3, 3, INV>(v);
    else if constexpr (R == 10) dft_pf<2, 5, INV>(v);
    else if constexpr (R == 12) dft_pf<3, 4, INV>(v);
    else if constexpr (R == 15) dft_pf<3, 5, INV>(v);
    else dft_ct<4, 4, INV>(v);
}

// Spectra that meet an alias fold: the S values of one column alias are consecutive
// (alias order, see starred_fft.hip)
template <int S>
__device__ __forceinline__ void alias_load(const float2 *__restrict__ X, int at, float2 (&v)[S])
{
    if constexpr (S == 2) {
        const float4 q = *reinterpret_cast<const float4 *>(X + at);  // (at is even: 16-byte aligned)
        v[0] = make_float2(q.x, q.y);
        v[1] = make_float2(q.z, q.w);
    } else {
        #pragma unroll
        for (int a = 0; a < S; ++a) v[a] = X[at + a];
    }
}

}  // namespace starred
