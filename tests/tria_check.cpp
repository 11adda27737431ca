// Host build of the library's FP64 Tria (lq_rows).  Prints, for the 5 x 10
// matrix [X, e Y] with X and Y lower (X of positive diagonal: a factor, and the
// process noise beside it) and for several e, the rms error of the Gram of the
// result in units of 2^-53: the library's, and that of the textbook sweep with
// the pivot a - r, two divisions and a rounded root.  With the argument "small":
// how far Tria(2^-500 A) is from 2^-500 Tria(A) (largest entry's difference, in
// units of 2^-53 of the row's norm), and Tria of the diagonal +-1e-200, 1e-3.
// Test infrastructure: compiled and run by tests/test_tria_cpu.py.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>

#if !defined(__HIP_DEVICE_COMPILE__)
// host stand-ins for the device builtins: reciprocal estimates of 24 bits
static inline double host_est(double x)
{
    int e;
    const double m = std::frexp(x, &e);
    return std::isfinite(x) ? std::ldexp((double)(float)m, e) : x;
}
static inline int host_frexp_exp(double x)
{
    int e;
    std::frexp(x, &e);
    return e;
}
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_rcp(x) host_est(1.0 / (x))
#define __builtin_amdgcn_rsq(x) host_est(1.0 / std::sqrt(x))
#define __builtin_amdgcn_frexp_expf(x) host_frexp_exp((double)(x))
#define __builtin_amdgcn_frexp_exp(x) host_frexp_exp(x)
#define __builtin_amdgcn_ldexpf(x, e) std::ldexp((float)(x), e)
#define __builtin_amdgcn_ldexp(x, e) std::ldexp((double)(x), e)
#endif

#include "../paper_2207_00426_amd/csrc/device_math.hpp"

constexpr int N = 5;

// uniform in (0, 1), and a sum of them near a normal
static double uniform()
{
    static unsigned long long s = 88172645463325252ull;
    s ^= s << 13;
    s ^= s >> 7;
    s ^= s << 17;
    return ((double)(s >> 11) + 0.5) * 0x1p-53;
}
static double normal()
{
    double x = -6.0;
    for (int i = 0; i < 12; ++i)
        x += uniform();
    return x;
}

static void draw(double e, double (&X)[N][N], double (&Y)[N][N])
{
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < N; ++j) {
            X[i][j] = j < i ? normal() : j == i ? std::fabs(normal()) + 0.3 : 0.0;
            Y[i][j] = j <= i ? e * normal() : 0.0;
        }
}

static void textbook(const double (&X)[N][N], const double (&Y)[N][N], double (&L)[N][N])
{
    double A[N][2 * N];
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < N; ++j) {
            A[i][j] = X[i][j];
            A[i][N + j] = Y[i][j];
        }
    for (int i = 0; i < N; ++i) {
        double s = 0.0;
        for (int j = i + 1; j < 2 * N; ++j)
            s = std::fma(A[i][j], A[i][j], s);
        const double a = A[i][i], r = std::sqrt(std::fma(a, a, s));
        if (s > 0.0) {
            const double v0 = a > 0.0 ? -s / (a + r) : a - r, tau = -1.0 / (r * v0);
            for (int k = i + 1; k < N; ++k) {
                double w = v0 * A[k][i];
                for (int j = i + 1; j < 2 * N; ++j)
                    w = std::fma(A[k][j], A[i][j], w);
                A[k][i] = std::fma(-tau * w, v0, A[k][i]);
                for (int j = i + 1; j < 2 * N; ++j)
                    A[k][j] = std::fma(-tau * w, A[i][j], A[k][j]);
            }
        }
        for (int j = 0; j <= i; ++j)
            L[i][j] = j < i ? A[i][j] : r;
    }
}

// |L L^T - X X^T - Y Y^T| / |X X^T + Y Y^T|, Frobenius, squared
static double gram_err(const double (&X)[N][N], const double (&Y)[N][N], const double (&L)[N][N])
{
    long double num = 0, den = 0;
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < N; ++j) {
            long double a = 0, b = 0;
            for (int t = 0; t < N; ++t) {
                a += (long double)X[i][t] * X[j][t] + (long double)Y[i][t] * Y[j][t];
                if (t <= i && t <= j)
                    b += (long double)L[i][t] * L[j][t];
            }
            num += (a - b) * (a - b);
            den += a * a;
        }
    return (double)(num / den);
}

static void small()
{
    const double f = 0x1p-500;
    double worst = 0.0;
    for (int k = 0; k < 1000; ++k) {
        double X[N][N], Y[N][N], L[N][N], l[N][N];
        draw(1.0, X, Y);
        pss::tria_dense_lower(X, Y, L);
        for (int i = 0; i < N; ++i)
            for (int j = 0; j < N; ++j) {
                X[i][j] *= f;
                Y[i][j] *= f;
            }
        pss::tria_dense_lower(X, Y, l);
        for (int i = 0; i < N; ++i) {
            double nr = 0.0;
            for (int j = 0; j <= i; ++j)
                nr += L[i][j] * L[i][j];
            for (int j = 0; j <= i; ++j) {
                const double d = std::fabs(l[i][j] / f - L[i][j]) / std::sqrt(nr) * 0x1p53;
                worst = d <= worst ? worst : d; // keeps a NaN
            }
        }
    }
    std::printf("%g\n", worst);
    double D[N][N] = {}, Z[N][N] = {}, L[N][N];
    for (int i = 0; i < N; ++i)
        D[i][i] = i == 2 ? 1e-3 : i == 1 ? -1e-200 : 1e-200;
    pss::tria_dense_lower(D, Z, L);
    for (int i = 0; i < N; ++i)
        std::printf("%.17g ", L[i][i]);
    std::printf("\n");
}

int main(int argc, char **)
{
    if (argc > 1) {
        small();
        return 0;
    }
    const int reps = 20000;
    for (double e : {1.0, 1e-1, 1e-2, 1e-4, 1e-6, 1e-8, 0.0}) {
        double lib = 0.0, ref = 0.0;
        for (int k = 0; k < reps; ++k) {
            double X[N][N], Y[N][N], L[N][N];
            draw(e, X, Y);
            pss::tria_dense_lower(X, Y, L);
            lib += gram_err(X, Y, L);
            textbook(X, Y, L);
            ref += gram_err(X, Y, L);
        }
        std::printf("%g %.4f %.4f\n", e, std::sqrt(lib / reps) * 0x1p53,
                    std::sqrt(ref / reps) * 0x1p53);
    }
    return 0;
}
