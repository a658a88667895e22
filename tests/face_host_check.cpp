// Host check of the closed forms of the RHD face dissipation (compiled for the CPU from
// the device header): face_eigen_columns against the numerically formed columns
// (face_eigen_columns_gram) on random face states from near rest to fast flow, cold to
// hot, with velocities along and across the normal; weno_jump<P> against the two
// one-sided weno3 / weno5 / weno7 values on smooth, random, constant and jump data.
// Tolerances: columns 1e-10 of the column (the numerical route, run in extended
// precision, inverts a Gram matrix whose condition grows like W^4, W <= 4 here); jumps 64 roundings of the largest value
// (the one-sided values are rounded at that level) plus 1e-10 of the jump.
#include "es_common.h"
#include <cmath>
#include <cstdio>
#include <random>
#undef __device__
#define __device__
#undef __forceinline__
#define __forceinline__ inline
#define ES_OPCOUNT_HOST 1
// the header's scalar functions in extended precision, for the numerical route
namespace es {
inline long double frcp(long double x) { return 1.0L / x; }
inline long double frsqrt(long double x) { return 1.0L / std::sqrt(x); }
inline long double psqrt(long double x) { return std::sqrt(x); }
inline long double xsqrt(long double x) { return std::sqrt(x); }
inline long double xexp(long double x) { return std::exp(x); }
inline long double xlog(long double x) { return std::log(x); }
inline long double fabs(long double x) { return std::fabs(x); }
inline double fabs(double x) { return std::fabs(x); }
inline long double fmax(long double x, long double y) { return std::fmax(x, y); }
inline double fmax(double x, double y) { return std::fmax(x, y); }
}  // namespace es
#include "es_rhd.h"
using es::face_eigen_columns;
using es::face_eigen_columns_gram;
using es::weno3;
using es::weno5;
using es::weno7;
using es::weno_jump;

template <int DIM>
int run_columns(std::mt19937_64& rng, int trials) {
    constexpr int M = DIM + 2;
    std::uniform_real_distribution<double> U(0.0, 1.0);
    double worst = 0.0;
    for (int t = 0; t < trials; ++t) {
        const double G = 1.1 + 0.8 * U(rng), c0 = G / (G - 1.0), c1 = 1.0 / (G - 1.0);
        const double rho = std::pow(10.0, 4.0 * U(rng) - 2.0), p = std::pow(10.0, 4.0 * U(rng) - 2.0), beta = rho / p;
        const double scale = t % 4 == 0 ? 0.0 : (t % 4 == 1 ? 1e-3 : (t % 4 == 2 ? 0.5 : 2.2));
        double u[3] = {0.0, 0.0, 0.0}, uu = 0.0;
        for (int k = 0; k < DIM; ++k) u[k] = scale * 2.0 * (U(rng) - 0.5);
        if (t % 5 == 0) u[0] = 0.0;
        if (t % 7 == 0) for (int k = 1; k < DIM; ++k) u[k] = 0.0;
        for (int k = 0; k < DIM; ++k) uu += u[k] * u[k];
        const double W = std::sqrt(1.0 + uu);
        double V[M];
        V[0] = c0 + std::log(rho) + std::log(beta) * c1 + beta;
        for (int k = 0; k < DIM; ++k) V[1 + k] = beta * u[k];
        V[M - 1] = -beta * W;
        const double at = 2.0 * (U(rng) - 0.5), L = 0.5 + U(rng);
        long double Vx[M], B[M][M];
        double A[M][M];
        for (int c = 0; c < M; ++c) Vx[c] = V[c];
        const double la = face_eigen_columns<DIM>(G, V, V, at, L, [&](const double* r, int q) { for (int c = 0; c < M; ++c) A[q][c] = r[c]; });
        const long double lb = face_eigen_columns_gram<DIM, long double>(
            G, Vx, Vx, at, L, [&](const long double* r, int q) { for (int c = 0; c < M; ++c) B[q][c] = r[c]; });
        worst = std::fmax(worst, (double)(std::fabs(la - lb) / std::fabs(lb)));
        for (int q = 0; q < M; ++q) {
            double n = 0.0, e = 0.0;
            for (int c = 0; c < M; ++c) {
                n = std::fmax(n, (double)std::fabs(B[q][c]));
                e = std::fmax(e, (double)std::fabs(A[q][c] - B[q][c]));
            }
            worst = std::fmax(worst, e / n);
        }
    }
    printf("DIM=%d: worst relative difference of the columns and lambda^ %.3e\n", DIM, worst);
    return worst < 1e-10 ? 0 : 1;
}

template <int P>
int run_weno(std::mt19937_64& rng, int trials) {
    std::uniform_real_distribution<double> U(0.0, 1.0);
    double worst = 0.0;
    const double eps = 1e-6;
    for (int t = 0; t < trials; ++t) {
        double v[2 * P];
        const double base = 10.0 * (U(rng) - 0.5), amp = std::pow(10.0, 4.0 * U(rng) - 3.0), h = 0.3 * U(rng);
        for (int k = 0; k < 2 * P; ++k)
            v[k] = t % 4 == 0 ? base + amp * std::sin(h * k + base)
                 : t % 4 == 1 ? base + amp * (U(rng) - 0.5)
                 : t % 4 == 2 ? base : base + (k < P ? 0.0 : amp);
        double l, r;
        if constexpr (P == 2) { l = weno3(v[0], v[1], v[2], eps); r = weno3(v[3], v[2], v[1], eps); }
        else if constexpr (P == 3) { l = weno5(v[0], v[1], v[2], v[3], v[4], eps); r = weno5(v[5], v[4], v[3], v[2], v[1], eps); }
        else { l = weno7(v[0], v[1], v[2], v[3], v[4], v[5], v[6], eps); r = weno7(v[7], v[6], v[5], v[4], v[3], v[2], v[1], eps); }
        const double want = r - l, got = weno_jump<P, double>(v, eps);
        if (t % 4 == 2 && got != 0.0) return printf("P=%d: constant data give a jump\n", P), 1;
        double big = 0.0;
        for (int k = 0; k < 2 * P; ++k) big = std::fmax(big, std::fabs(v[k]));
        worst = std::fmax(worst, std::fabs(got - want) / (64.0 * 2.22e-16 * big + 1e-10 * std::fabs(want)));
    }
    printf("P=%d: worst jump difference %.3f of its bound\n", P, worst);
    return worst < 1.0 ? 0 : 1;
}

int main() {
    std::mt19937_64 rng(11);
    return run_columns<2>(rng, 20000) + run_columns<3>(rng, 20000) + run_weno<2>(rng, 20000) + run_weno<3>(rng, 20000) +
           run_weno<4>(rng, 20000);
}
