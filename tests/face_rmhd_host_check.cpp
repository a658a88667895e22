// Host check of the closed-form eigen-structure of the RMHD face (compiled for the CPU from
// the device header), against the matrices A0 = dU/dV and H = dF/dV + Phi' (dB_n/dV)^T of
// the Godunov-Powell modified system (derivatives by complex steps in extended precision):
//   R R^T = A0,  R Lambda R^T = H,
// and, where eigenvalues fall into groups (a field along or across the normal, no field, rest,
// each exactly or with perturbations from 1e-3 down to denormals), the canonical order of each
// group: the seed that a column belongs to has no component along the later columns.
// Tolerances, for states with W <= 2.5 and rho, p, |b| within a decade or two: 1e-10 of the
// norm of A0 (rounding times the square of the condition of the tetrad and the Cholesky
// factor, about 1e5; |lambda| <= 1); H with groups 1e-5 of it (eigenvalues within 1e-6, up to 8
// in a chain, are taken as one, and A0 carries that difference into H); seeds 1e-9 of their norm (rounding times the root of the condition of A0).
#include "es_common.h"
#include <cmath>
#include <complex>
#include <cstdio>
#include <random>
#undef __device__
#define __device__
#undef __forceinline__
#define __forceinline__ inline
#define ES_OPCOUNT_HOST 1
#include "es_rmhd.h"

typedef std::complex<long double> C;

static void conserved(long double G, const C* V, C* U, C* F, C* Phi) {
    const C beta = std::sqrt(V[4] * V[4] - V[1] * V[1] - V[2] * V[2] - V[3] * V[3]);
    const C W = -V[4] / beta;
    C u[3], b[3], b0 = 0.0L, bb = 0.0L;
    for (int k = 0; k < 3; ++k) {
        u[k] = V[1 + k] / beta;
        b[k] = V[5 + k] / beta;
        b0 += u[k] * b[k] / W;
        bb += b[k] * b[k];
    }
    bb -= b0 * b0;
    const C rho = std::exp(V[0] - G / (G - 1.0L) - std::log(beta) / (G - 1.0L) - beta), p = rho / beta;
    const C w = rho + G / (G - 1.0L) * p + bb, pt = p + 0.5L * bb;
    U[0] = rho * W;
    F[0] = rho * u[0];
    U[4] = w * W * W - pt - b0 * b0;
    for (int k = 0; k < 3; ++k) {
        U[1 + k] = w * W * u[k] - b0 * b[k];
        F[1 + k] = w * u[0] * u[k] - b[0] * b[k] + (k == 0 ? pt : C(0.0L));
        U[5 + k] = W * b[k] - b0 * u[k];
        F[5 + k] = u[0] * b[k] - b[0] * u[k];
    }
    F[4] = U[1];
    // phi = V . Phi = beta b^0 ... : Phi = (0, B / W^2 + v (v.B), v.B, v)
    const C vB = b0 / W;
    Phi[0] = 0.0L;
    Phi[4] = vB;
    for (int k = 0; k < 3; ++k) {
        Phi[1 + k] = U[5 + k] / (W * W) + vB * u[k] / W;
        Phi[5 + k] = u[k] / W;
    }
}

int main() {
    std::mt19937_64 rng(7);
    std::uniform_real_distribution<double> X(0.0, 1.0);
    double worst[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    int groups = 0;
    for (int t = 0; t < 24000; ++t) {
        const double G = 1.2 + 0.7 * X(rng), c0 = G / (G - 1.0), c1 = 1.0 / (G - 1.0);
        const double rho = std::pow(10.0, 2.0 * X(rng) - 1.0), p = std::pow(10.0, 2.0 * X(rng) - 1.0), beta = rho / p;
        const double us = t % 3 == 0 ? 0.0 : (t % 3 == 1 ? 0.1 : 1.2), bs = std::pow(10.0, 1.5 * X(rng) - 1.0);
        double u[3], b[3], uu = 0.0;
        for (int k = 0; k < 3; ++k) {
            u[k] = us * 2.0 * (X(rng) - 0.5);
            b[k] = bs * 2.0 * (X(rng) - 0.5);
        }
        const int kind = (t / 3) % 6;
        if (kind == 1) b[1] = b[2] = 0.0;
        if (kind == 2) b[0] = 0.0;
        if (kind == 3) b[0] = b[1] = b[2] = 0.0;
        if (kind == 4) u[1] = u[2] = b[1] = b[2] = 0.0;
        if (kind == 5) u[0] = u[1] = b[0] = 0.0;
        if (kind && (t / 18) % 2) {
            // about the degenerate state, at any scale
            const int q = (t / 36) % 40;
            const double e = std::pow(10.0, -3.0 - (q < 20 ? q : 16.0 * (q - 18)));
            for (int k = 0; k < 3; ++k) {
                u[k] += (X(rng) < 0.7) * e * (X(rng) - 0.5);
                b[k] += (X(rng) < 0.7) * e * (X(rng) - 0.5);
            }
        }
        for (int k = 0; k < 3; ++k) uu += u[k] * u[k];
        double V[8] = {c0 + std::log(rho) + std::log(beta) * c1 + beta, 0, 0, 0, -beta * std::sqrt(1.0 + uu), 0, 0, 0};
        for (int k = 0; k < 3; ++k) {
            V[1 + k] = beta * u[k];
            V[5 + k] = beta * b[k];
        }
        // A0 and H
        long double A0[8][8], H[8][8];
        for (int j = 0; j < 8; ++j) {
            C Vc[8], U[8], F[8], Phi[8];
            const long double h = 1e-40L;
            for (int c = 0; c < 8; ++c) Vc[c] = C(V[c], c == j ? h : 0.0L);
            conserved(G, Vc, U, F, Phi);
            for (int c = 0; c < 8; ++c) {
                A0[c][j] = U[c].imag() / h;
                H[c][j] = (F[c].imag() + Phi[c].real() * U[5].imag()) / h;
            }
        }
        double mu[6], Z[6][6], R[8][8], lam[8];
        bool grouped;
        const double vn = -V[1] / V[4];
        es::rmhd_face_modes(G, c0, c1, V, mu, Z);
        es::rmhd_face_speed(V, mu, 0.1, 1.0, grouped);
        es::rmhd_face_columns(G, c0, c1, V, mu, Z, grouped, [&](int k, const double* r) {
            lam[k] = k < 6 ? vn + mu[k < 6 ? k : 0] : vn;
            for (int c = 0; c < 8; ++c) R[c][k] = r[c];
        });
        groups += grouped;
        long double nA = 0.0L, eA = 0.0L, eH = 0.0L;
        for (int i = 0; i < 8; ++i)
            for (int j = 0; j < 8; ++j) {
                long double a = 0.0L, h = 0.0L;
                for (int k = 0; k < 8; ++k) {
                    a += (long double)R[i][k] * R[j][k];
                    h += (long double)R[i][k] * lam[k] * R[j][k];
                }
                nA += A0[i][j] * A0[i][j];
                eA += (a - A0[i][j]) * (a - A0[i][j]);
                eH += (h - H[i][j]) * (h - H[i][j]);
            }
        auto note = [&](int m, double e) { worst[m] = e <= worst[m] ? worst[m] : (e < 1.0 ? e : 1.0); };
        note(grouped, (double)std::sqrt(eA / nA));
        note(2 + grouped, (double)std::sqrt(eH / nA));
        if (!grouped) continue;
        int id[8];
        for (int k = 0; k < 8; ++k) id[k] = k;
        for (int s = 0; s < 8; ++s)
            for (int j = 0; j < 8; ++j)
                for (int k = 0; k < 8; ++k)
                    if (std::fabs(lam[j] - lam[k]) <= es::GROUP_TOL) id[j] = id[k] = id[j] < id[k] ? id[j] : id[k];
        for (int g = 0; g < 8; ++g) {
            if (id[g] != g) continue;
            bool placed[8] = {};
            for (int q = 0; q < 8; ++q) {
                const int seed = id[6] == g ? (q == 0 ? 0 : (q == 1 ? 5 : (q < 6 ? q - 1 : q))) : q;
                // x = A0^{-1} e_seed
                long double M[8][9];
                for (int i = 0; i < 8; ++i) {
                    for (int j = 0; j < 8; ++j) M[i][j] = A0[i][j];
                    M[i][8] = i == seed;
                }
                for (int c = 0; c < 8; ++c) {
                    for (int i = c + 1; i < 8; ++i)
                        for (int j = 8; j >= c; --j) M[i][j] -= M[i][c] / M[c][c] * M[c][j];
                }
                long double x[8];
                for (int i = 7; i >= 0; --i) {
                    x[i] = M[i][8];
                    for (int j = i + 1; j < 8; ++j) x[i] -= M[i][j] * x[j];
                    x[i] /= M[i][i];
                }
                const long double n = std::sqrt(x[seed]);
                int at = -1;
                bool unsure = false;
                double later = 0.0;
                for (int k = 0; k < 8; ++k) {
                    if (id[k] != g || placed[k]) continue;
                    long double y = 0.0L;
                    for (int c = 0; c < 8; ++c) y += R[c][k] * x[c];
                    const double rel = (double)(std::fabs(y) / n);
                    if (at < 0) {
                        at = k;
                        if (rel > 0.5 * es::SEED_TOL && rel < 2.0 * es::SEED_TOL) unsure = true;
                        if (rel <= 0.5 * es::SEED_TOL) break;
                        placed[k] = true;
                    } else {
                        later = rel <= later ? later : (rel < 1.0 ? rel : 1.0);
                    }
                }
                if (unsure) break;
                note(4, later);
            }
        }
    }
    printf("RR^T %.2e (groups %.2e), R Lambda R^T %.2e (groups %.2e), seeds %.2e; %d faces with groups\n", worst[0],
           worst[1], worst[2], worst[3], worst[4], groups);
    return worst[0] < 1e-10 && worst[1] < 1e-10 && worst[2] < 1e-10 && worst[3] < 1e-5 && worst[4] < 1e-9 ? 0 : 1;
}
