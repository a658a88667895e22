// Host check of the hand-written RMHD backward sweeps (compiled for the CPU from the device
// headers): pair_vjp_rmhd and node_vjp_rmhd against forward-mode dual-number derivatives of
// pair_flux_rmhd, on random pairs and on small jumps (the series branch of the logarithmic
// mean), 2D and 3D; and weno_jump_grad against dual numbers through the one-sided values.
// Tolerance 1e-11 of the largest cotangent: rounding (a few hundred operations) times the
// largest ratio of a term to its sum at these states, about 1e3.  (WENO gradients: of the
// larger of it and one, the weights' derivatives of the oracle being up to 1e3 before they
// cancel.)
#include "es_common.h"
#include <cmath>
#include <cstdio>
#include <random>
#undef __device__
#define __device__
#undef __forceinline__
#define __forceinline__ inline
#define ES_OPCOUNT_HOST 1
#include "es_pair_vjp_rmhd.h"
using namespace es;

static NodeQM node(const double* P) {
    NodeQM q;
    double uu = 0.0, uB = 0.0;
    for (int k = 0; k < 3; ++k) {
        q.u[k] = P[1 + k];
        q.B[k] = P[5 + k];
        uu += q.u[k] * q.u[k];
        uB += q.u[k] * q.B[k];
    }
    q.rho = P[0];
    q.beta = P[0] / P[4];
    q.lr = std::log(q.rho);
    q.lb = std::log(q.beta);
    q.W = std::sqrt(1.0 + uu);
    q.b0 = uB;
    for (int k = 0; k < 3; ++k) q.b[k] = (q.B[k] + uB * q.u[k]) / q.W;
    return q;
}

template <int DIM>
int run(std::mt19937_64& rng, bool small) {
    std::uniform_real_distribution<double> X(0.0, 1.0);
    using D = Dual<16>;
    const double G = 5.0 / 3.0;
    double worst = 0.0;
    for (int t = 0; t < 5000; ++t) {
        double P[2][8], al[DIM + 1], ar[DIM + 1], w[8];
        for (int c = 0; c < 8; ++c) P[0][c] = c == 0 || c == 4 ? 0.1 + X(rng) : 2.0 * (X(rng) - 0.5);
        for (int c = 0; c < 8; ++c)
            P[1][c] = small ? P[0][c] * (1.0 + 1e-3 * (X(rng) - 0.5)) : (c == 0 || c == 4 ? 0.1 + X(rng) : 2.0 * (X(rng) - 0.5));
        for (int c = 0; c <= DIM; ++c) { al[c] = X(rng) - 0.5; ar[c] = X(rng) - 0.5; }
        for (int c = 0; c < 8; ++c) w[c] = X(rng) - 0.5;
        D Pd[2][8], F[8];
        for (int s = 0; s < 2; ++s)
            for (int c = 0; c < 8; ++c) Pd[s][c] = D::seed(P[s][c], 8 * s + c);
        const NodeRMHDT<D> l = node_rmhd<D>(G, Pd[0], xlog(Pd[0][0]), xlog(Pd[0][0] / Pd[0][4]));
        const NodeRMHDT<D> r = node_rmhd<D>(G, Pd[1], xlog(Pd[1][0]), xlog(Pd[1][0] / Pd[1][4]));
        double Jt, Bt;
        pair_flux_rmhd<DIM, D, D>(G, l, r, al, ar, F, Jt, Bt);
        const NodeQM ql = node(P[0]), qr = node(P[1]);
        double g[2][num_q<DIM>()], gP[2][8], want[16], big = 0.0;
        pair_vjp_rmhd<DIM>(G, ql, qr, al, ar, w, g[0], g[1]);
        node_vjp_rmhd<DIM>(ql, g[0], gP[0]);
        node_vjp_rmhd<DIM>(qr, g[1], gP[1]);
        for (int k = 0; k < 16; ++k) {
            want[k] = 0.0;
            for (int c = 0; c < 8; ++c) want[k] += w[c] * F[c].d[k];
            big = std::fmax(big, std::fabs(want[k]));
        }
        for (int k = 0; k < 16; ++k) {
            const double e = std::fabs(gP[k / 8][k % 8] - want[k]) / big;
            worst = e <= worst ? worst : (e < 1.0 ? e : 1.0);
        }
    }
    printf("pair DIM=%d %s: worst relative difference %.2e\n", DIM, small ? "small jumps" : "random", worst);
    return worst < 1e-11 ? 0 : 1;
}

template <int P>
int run_weno(std::mt19937_64& rng) {
    std::uniform_real_distribution<double> X(0.0, 1.0);
    using D = Dual<2 * P>;
    const double eps = 1e-6;
    double worst = 0.0;
    for (int t = 0; t < 5000; ++t) {
        double v[2 * P], g[2 * P];
        const double base = 4.0 * (X(rng) - 0.5), amp = std::pow(10.0, 3.0 * X(rng) - 3.0);
        for (int k = 0; k < 2 * P; ++k) v[k] = base + (t % 2 ? amp * std::sin(0.3 * k + base) : amp * (X(rng) - 0.5));
        const double jw = weno_jump_grad<P>(v, eps, g);
        D d[2 * P];
        for (int k = 0; k < 2 * P; ++k) d[k] = D::seed(v[k], k);
        // the one-sided values with the optimal weights d_k / (eps + beta_k)^2
        auto side = [&](bool right) {
            D x[2 * P - 1];
            for (int k = 0; k < 2 * P - 1; ++k) x[k] = right ? d[2 * P - 1 - k] : d[k];
            D q[P], be[P];
            double c[P];
            if (P == 3) {
                q[0] = (1.0 / 6.0) * (2.0 * x[0] - 7.0 * x[1] + 11.0 * x[2]);
                q[1] = (1.0 / 6.0) * (5.0 * x[2] - x[1] + 2.0 * x[3]);
                q[P - 1] = (1.0 / 6.0) * (2.0 * x[2] + 5.0 * x[3] - x[2 * P - 2]);
                const D t0 = x[0] - 2.0 * x[1] + x[2], t1 = x[1] - 2.0 * x[2] + x[3], t2 = x[2] - 2.0 * x[3] + x[2 * P - 2];
                const D s0 = x[0] - 4.0 * x[1] + 3.0 * x[2], s1 = x[1] - x[3], s2 = 3.0 * x[2] - 4.0 * x[3] + x[2 * P - 2];
                be[0] = (13.0 / 12.0) * t0 * t0 + 0.25 * s0 * s0;
                be[1] = (13.0 / 12.0) * t1 * t1 + 0.25 * s1 * s1;
                be[P - 1] = (13.0 / 12.0) * t2 * t2 + 0.25 * s2 * s2;
                c[0] = 0.1; c[1] = 0.6; c[P - 1] = 0.3;
            } else {
                q[0] = 0.5 * (3.0 * x[1] - x[0]);
                q[1] = 0.5 * (x[1] + x[2]);
                be[0] = (x[1] - x[0]) * (x[1] - x[0]);
                be[1] = (x[2] - x[1]) * (x[2] - x[1]);
                c[0] = 1.0 / 3.0; c[1] = 2.0 / 3.0;
            }
            D S = D(0.0), v = D(0.0);
            for (int k = 0; k < P; ++k) {
                const D e = D(eps) + be[k], o = D(c[k]) / (e * e);
                S = S + o;
                v = v + o * q[k];
            }
            return v / S;
        };
        const D j = side(true) - side(false);
        double big = 1.0;
        for (int k = 0; k < 2 * P; ++k) big = std::fmax(big, std::fabs(j.d[k]));
        double e = std::fabs(jw - j.v) / (std::fabs(base) + amp + big);
        for (int k = 0; k < 2 * P; ++k) e = std::fmax(e, std::fabs(g[k] - j.d[k]) / big);
        worst = e <= worst ? worst : (e < 1.0 ? e : 1.0);
    }
    printf("weno P=%d: worst relative difference %.2e\n", P, worst);
    return worst < 1e-11 ? 0 : 1;
}

int main() {
    std::mt19937_64 rng(5);
    return run<2>(rng, false) + run<3>(rng, false) + run<2>(rng, true) + run<3>(rng, true) + run_weno<2>(rng) +
           run_weno<3>(rng);
}
