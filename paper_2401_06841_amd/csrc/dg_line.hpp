// dg_line.hpp -- evaluation and moments along one line of Gauss points.
//
// The volume and face kernels work line by line: the expansion of a cell is first reduced to
// the K+1 (or fewer) coefficients of one line of K+1 points (one multiply-add per mode), the
// points of the line then cost 1D polynomials only, and what was formed at the points goes back
// through the 1D moments of the line.  Against the 3D basis tables at every point that is, at
// degree 2, 93 instead of 270 multiply-adds per variable for the values at the 27 points (at
// degree 3, 416 instead of 1,280 for 64), and the constants of a line are the same for every
// line: they stay in scalar registers instead of being loaded per point.  The Gauss points are
// symmetric, so even and odd parts of two mirrored points are formed once.
//
// Every operation is an explicit fused multiply-add, product or sum with no other contraction:
// all kernels that evaluate the same line get the same bits.
#pragma once

#include <hip/hip_runtime.h>

#include "dg_basis.hpp"

namespace dg {

// square root by Newton's iteration, for constants formed at compile time
constexpr double csqrt(double a)
{
    double x = a < 1.0 ? 1.0 : a;
    for (int i = 0; i < 64; ++i) x = 0.5 * (x + a / x);
    return x;
}

// the K+1 Gauss-Legendre points (ascending), their weights, and Lt_n(x_t) (n <= K)
template <int K>
struct Gauss {
    double x[K + 1], w[K + 1], P[K + 1][K + 1];     // P[n][t]
};

template <int K>
constexpr Gauss<K> make_gauss()
{
    Gauss<K> G{};
    if constexpr (K == 1) {
        G.x[1] = 1.0 / csqrt(3.0);
        G.x[0] = -G.x[1];
        G.w[0] = G.w[1] = 1.0;
    } else if constexpr (K == 2) {
        G.x[2] = csqrt(0.6);
        G.x[0] = -G.x[2];
        G.w[0] = G.w[2] = 5.0 / 9.0;
        G.w[1] = 8.0 / 9.0;
    } else {
        G.x[3] = csqrt(3.0 / 7.0 + 2.0 / 7.0 * csqrt(1.2));
        G.x[2] = csqrt(3.0 / 7.0 - 2.0 / 7.0 * csqrt(1.2));
        G.x[0] = -G.x[3];
        G.x[1] = -G.x[2];
        G.w[0] = G.w[3] = (18.0 - csqrt(30.0)) / 36.0;
        G.w[1] = G.w[2] = (18.0 + csqrt(30.0)) / 36.0;
    }
    for (int t = 0; t <= K; ++t) {
        const double x = G.x[t];
        const double p[4] = {1.0, x, 0.5 * (3.0 * x * x - 1.0), 0.5 * (5.0 * x * x - 3.0) * x};
        for (int n = 0; n <= K; ++n) G.P[n][t] = csqrt(2.0 * n + 1.0) * p[n];
    }
    return G;
}

// values v[t] = sum_{n < N} c[n] Lt_n(x_t) at the K+1 points
template <int K, int N, typename T>
__device__ __forceinline__ void line_eval(const T (&c)[N], T (&v)[K + 1])
{
#pragma clang fp contract(off)
    constexpr Gauss<K> G = make_gauss<K>();
    static_assert(N >= 1 && N <= K + 1, "line coefficients");
    if constexpr (N == 1) {
#pragma unroll
        for (int t = 0; t <= K; ++t) v[t] = c[0];
    } else if constexpr (K == 1) {
        // Lt_1(x) = sqrt(3) x = +-1
        v[0] = c[0] - c[1];
        v[1] = c[0] + c[1];
    } else if constexpr (K == 2) {
        T e = c[0], mid = c[0];
        if constexpr (N > 2) {
            e = fma(T(G.P[2][2]), c[2], c[0]);
            mid = fma(T(G.P[2][1]), c[2], c[0]);
        }
        v[0] = fma(T(-G.P[1][2]), c[1], e);
        v[1] = mid;
        v[2] = fma(T(G.P[1][2]), c[1], e);
    } else {
#pragma unroll
        for (int t = 2; t <= 3; ++t) {
            T e = c[0];
            if constexpr (N > 2) e = fma(T(G.P[2][t]), c[2], c[0]);
            if constexpr (N > 3) {
                const T o = fma(T(G.P[3][t]), c[3], T(G.P[1][t]) * c[1]);
                v[3 - t] = e - o;
                v[t] = e + o;
            } else {
                v[3 - t] = fma(T(-G.P[1][t]), c[1], e);
                v[t] = fma(T(G.P[1][t]), c[1], e);
            }
        }
    }
}

// moments m[n] = sum_t w_t Lt_n(x_t) f[t], n < N
template <int K, int N, typename T>
__device__ __forceinline__ void line_moments(const T (&f)[K + 1], T (&m)[N])
{
#pragma clang fp contract(off)
    constexpr Gauss<K> G = make_gauss<K>();
    static_assert(N >= 1 && N <= K + 1, "line moments");
    if constexpr (K == 1) {
        m[0] = f[0] + f[1];
        if constexpr (N > 1) m[1] = f[1] - f[0];
    } else if constexpr (K == 2) {
        const T s = f[0] + f[2];
        m[0] = fma(T(G.w[1]), f[1], T(G.w[0]) * s);
        if constexpr (N > 1) m[1] = T(G.w[2] * G.P[1][2]) * (f[2] - f[0]);
        if constexpr (N > 2) m[2] = fma(T(G.w[1] * G.P[2][1]), f[1], T(G.w[2] * G.P[2][2]) * s);
    } else {
        const T sa = f[0] + f[3], sb = f[1] + f[2];
        m[0] = fma(T(G.w[3]), sa, T(G.w[2]) * sb);
        if constexpr (N > 2) m[2] = fma(T(G.w[3] * G.P[2][3]), sa, T(G.w[2] * G.P[2][2]) * sb);
        if constexpr (N > 1) {
            const T da = f[3] - f[0], db = f[2] - f[1];
            m[1] = fma(T(G.w[3] * G.P[1][3]), da, T(G.w[2] * G.P[1][2]) * db);
            if constexpr (N > 3) m[3] = fma(T(G.w[3] * G.P[3][3]), da, T(G.w[2] * G.P[3][2]) * db);
        }
    }
}

// line_moments in steps of mirrored points, to hold fewer point values at a time: step P = 0, 1, ..
// (2 P <= K) adds the points P and K - P, with values lo and hi (the middle point of an even K:
// hi, lo unused), to m; step 0 sets m
template <int K, int N, int P, typename T>
__device__ __forceinline__ void line_moments_step(T lo, T hi, T (&m)[N])
{
#pragma clang fp contract(off)
    constexpr Gauss<K> G = make_gauss<K>();
    constexpr bool MID = 2 * P == K;
    const T s = MID ? hi : lo + hi, d = MID ? T(0) : hi - lo;
#pragma unroll
    for (int n = 0; n < N; ++n) {
        if (MID && (n & 1)) continue;
        const T w = T(G.w[K - P] * G.P[n][K - P]);
        if (P == 0) m[n] = w * ((n & 1) ? d : s);
        else m[n] = fma(w, (n & 1) ? d : s, m[n]);
    }
}

// the moments of f against the derivatives, d[n] = sum_t w_t Lt_n'(x_t) f[t] (d[0] = 0), from
// f's moments below degree K: Lt_n' = sum over j = n-1, n-3, ... of sqrt((2n+1)(2j+1)) Lt_j
template <int K, typename T>
__device__ __forceinline__ void line_derivative(const T (&m)[K], T (&d)[K + 1])
{
#pragma clang fp contract(off)
    d[0] = T(0);
    d[1] = T(__builtin_sqrt(3.0)) * m[0];
    if constexpr (K > 1) d[2] = T(__builtin_sqrt(15.0)) * m[1];
    if constexpr (K > 2) d[3] = fma(T(__builtin_sqrt(35.0)), m[2], T(__builtin_sqrt(7.0)) * m[0]);
}

// coefficients along z of the line of volume points (t_x, t_y), c[n] = sum of the modes with z
// degree n, from the line's 2D basis values phi2 (the F2 row of r = t_x + (K+1) t_y); modes of
// total degree < DEG only (N = DEG, at most K+1, coefficients)
template <typename T, int K, int DEG, typename W, typename B>
__device__ __forceinline__ void line_coefficients(const W &w, const B &phi2, T (&c)[DEG])
{
#pragma clang fp contract(off)
#pragma unroll
    for (int n = 0; n < DEG; ++n) {
        T x = w[idx3(0, 0, n)];
#pragma unroll
        for (int s = 1; s < DEG - n; ++s)
#pragma unroll
            for (int b = 0; b <= s; ++b) x = fma(phi2[idx2(s - b, b)], w[idx3(s - b, b, n)], x);
        c[n] = x;
    }
}

// coefficients along the first tangential axis of the line of face points with second
// tangential point t2, c[p] = sum_q C[p, q] Lt_q(x_t2), from the 2D face coefficients C and
// the point's basis values p1 (the P1 row of t2)
template <typename T, int K, typename B>
__device__ __forceinline__ void face_line_coefficients(const T (&C)[(K + 1) * (K + 2) / 2], const B &p1, T (&c)[K + 1])
{
#pragma clang fp contract(off)
#pragma unroll
    for (int p = 0; p <= K; ++p) {
        T x = C[idx2(p, 0)];
#pragma unroll
        for (int q = 1; q <= K - p; ++q) x = fma(p1[q], C[idx2(p, q)], x);
        c[p] = x;
    }
}

}  // namespace dg
