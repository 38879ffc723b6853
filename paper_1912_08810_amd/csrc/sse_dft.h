// sse_dft.h -- small discrete Fourier transforms on register arrays of binary64
// complex values: sizes 2, 3, 4, 5 and 7 written out, larger ones as Cooley-Tukey
// products of two of them, with the twiddle factors as compile-time constants
// (trivial ones without a multiplication).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

namespace sse {

namespace dft {

constexpr double kPi2 = 1.57079632679489661923;  // pi / 2

// Taylor sums, for 0 <= x <= pi / 4 (the terms past x^24 are below 1e-25)
constexpr double taylor_sin(double x)
{
    double t = x, s = x;
    for (int n = 1; n <= 11; ++n) {
        t = -t * x * x / ((2 * n) * (2 * n + 1));
        s += t;
    }
    return s;
}
constexpr double taylor_cos(double x)
{
    double t = 1.0, s = 1.0;
    for (int n = 1; n <= 12; ++n) {
        t = -t * x * x / ((2 * n - 1) * (2 * n));
        s += t;
    }
    return s;
}
// cos and sin of 2 pi j / N, reduced to the first octant in integers
constexpr double quad_cos(int r, int N)
{
    return 2 * r > N ? taylor_sin(kPi2 * (double)(N - r) / N) : taylor_cos(kPi2 * (double)r / N);
}
constexpr double cos2pi(int j, int N)
{
    const int q = 4 * j / N, r = 4 * j - q * N;
    return q == 0 ? quad_cos(r, N) : q == 1 ? -quad_cos(N - r, N) : q == 2 ? -quad_cos(r, N)
                                                                          : quad_cos(N - r, N);
}
constexpr double sin2pi(int j, int N)
{
    const int q = 4 * j / N, r = 4 * j - q * N;
    return q == 0 ? quad_cos(N - r, N) : q == 1 ? quad_cos(r, N) : q == 2 ? -quad_cos(N - r, N)
                                                                         : -quad_cos(r, N);
}

__device__ __forceinline__ double2 add(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 sub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
// v times (c + i s)
__device__ __forceinline__ double2 cmul(double2 v, double c, double s)
{
    return make_double2(fma(v.x, c, -(v.y * s)), fma(v.x, s, v.y * c));
}
// v times i S
template <int S>
__device__ __forceinline__ double2 rot(double2 v)
{
    return S > 0 ? make_double2(-v.y, v.x) : make_double2(v.y, -v.x);
}

// v times exp(2 pi i S J / N)
template <int J, int N, int S>
__device__ __forceinline__ double2 twiddle(double2 v)
{
    constexpr int j = J % N;
    if constexpr (j == 0) {
        return v;
    } else if constexpr (4 * j == N) {
        return rot<S>(v);
    } else if constexpr (2 * j == N) {
        return make_double2(-v.x, -v.y);
    } else if constexpr (4 * j == 3 * N) {
        return rot<-S>(v);
    } else {
        constexpr double c = cos2pi(j, N), s = S * sin2pi(j, N);
        return cmul(v, c, s);
    }
}

template <int... I, typename F>
__device__ __forceinline__ void static_for_(std::integer_sequence<int, I...>, F f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F f)
{
    static_for_(std::make_integer_sequence<int, N>{}, f);
}

constexpr int first_factor(int N)
{
    return N % 4 == 0 && N > 4 ? 4 : N % 3 == 0 ? 3 : N % 2 == 0 ? 2 : N % 5 == 0 ? 5 : 7;
}

// In place: v[k] <- sum_n v[n] exp(2 pi i S n k / N).
template <int N, int S>
__device__ __forceinline__ void transform(double2 (&v)[N])
{
    if constexpr (N == 1) {
    } else if constexpr (N == 2) {
        const double2 a = v[0], b = v[1];
        v[0] = add(a, b);
        v[1] = sub(a, b);
    } else if constexpr (N == 3) {
        constexpr double s3 = S * sin2pi(1, 3);
        const double2 t = add(v[1], v[2]), d = sub(v[1], v[2]);
        const double2 m = make_double2(fma(-0.5, t.x, v[0].x), fma(-0.5, t.y, v[0].y));
        v[0] = add(v[0], t);
        v[1] = make_double2(fma(-s3, d.y, m.x), fma(s3, d.x, m.y));
        v[2] = make_double2(fma(s3, d.y, m.x), fma(-s3, d.x, m.y));
    } else if constexpr (N == 4) {
        const double2 a = add(v[0], v[2]), b = sub(v[0], v[2]);
        const double2 c = add(v[1], v[3]), d = rot<S>(sub(v[1], v[3]));
        v[0] = add(a, c);
        v[1] = add(b, d);
        v[2] = sub(a, c);
        v[3] = sub(b, d);
    } else if constexpr (N == 5) {
        constexpr double c1 = cos2pi(1, 5), c2 = cos2pi(2, 5);
        constexpr double s1 = S * sin2pi(1, 5), s2 = S * sin2pi(2, 5);
        const double2 p = add(v[1], v[4]), m = sub(v[1], v[4]);
        const double2 q = add(v[2], v[3]), n = sub(v[2], v[3]);
        const double2 a = make_double2(fma(c1, p.x, fma(c2, q.x, v[0].x)), fma(c1, p.y, fma(c2, q.y, v[0].y)));
        const double2 b = make_double2(fma(c2, p.x, fma(c1, q.x, v[0].x)), fma(c2, p.y, fma(c1, q.y, v[0].y)));
        const double2 e = make_double2(fma(s1, m.x, s2 * n.x), fma(s1, m.y, s2 * n.y));
        const double2 f = make_double2(fma(s2, m.x, -(s1 * n.x)), fma(s2, m.y, -(s1 * n.y)));
        v[0] = add(v[0], add(p, q));
        v[1] = make_double2(a.x - e.y, a.y + e.x);
        v[4] = make_double2(a.x + e.y, a.y - e.x);
        v[2] = make_double2(b.x - f.y, b.y + f.x);
        v[3] = make_double2(b.x + f.y, b.y - f.x);
    } else if constexpr (N == 7) {
        // pairs n, 7 - n: the factors' real parts act on sums, the imaginary ones on differences
        double2 p[3], m[3];
        static_for<3>([&](auto i) {
            p[i] = add(v[i + 1], v[6 - i]);
            m[i] = sub(v[i + 1], v[6 - i]);
        });
        const double2 z = v[0];
        v[0] = add(add(z, p[0]), add(p[1], p[2]));
        static_for<3>([&](auto i) {
            constexpr int k = decltype(i)::value + 1;
            constexpr double c1 = cos2pi(k, 7), c2 = cos2pi(2 * k % 7, 7), c3 = cos2pi(3 * k % 7, 7);
            constexpr double s1 = S * sin2pi(k, 7), s2 = S * sin2pi(2 * k % 7, 7), s3 = S * sin2pi(3 * k % 7, 7);
            const double2 a = make_double2(fma(c1, p[0].x, fma(c2, p[1].x, fma(c3, p[2].x, z.x))),
                                           fma(c1, p[0].y, fma(c2, p[1].y, fma(c3, p[2].y, z.y))));
            const double2 b = make_double2(fma(s1, m[0].x, fma(s2, m[1].x, s3 * m[2].x)),
                                           fma(s1, m[0].y, fma(s2, m[1].y, s3 * m[2].y)));
            v[k] = make_double2(a.x - b.y, a.y + b.x);
            v[7 - k] = make_double2(a.x + b.y, a.y - b.x);
        });
    } else {
        // n = B n1 + n2, k = k1 + A k2
        constexpr int A = first_factor(N), B = N / A;
        static_assert(A * B == N && A > 1 && B > 1, "unsupported transform size");
        static_for<B>([&](auto n2) {
            double2 t[A];
            static_for<A>([&](auto n1) { t[n1] = v[B * n1 + n2]; });
            transform<A, S>(t);
            static_for<A>([&](auto k1) {
                v[B * k1 + n2] = twiddle<decltype(n2)::value * decltype(k1)::value, N, S>(t[k1]);
            });
        });
        double2 o[N];
        static_for<A>([&](auto k1) {
            double2 t[B];
            static_for<B>([&](auto n2) { t[n2] = v[B * k1 + n2]; });
            transform<B, S>(t);
            static_for<B>([&](auto k2) { o[k1 + A * k2] = t[k2]; });
        });
        static_for<N>([&](auto i) { v[i] = o[i]; });
    }
}

}  // namespace dft

}  // namespace sse
