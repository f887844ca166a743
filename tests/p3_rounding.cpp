// Rounding of the P3 tetrahedron through its point orbits (P3Tet) and through
// the products of the tabulated derivatives, against extended precision, over
// nodal fields and coefficients of several kinds. Prints one line per
// combination: physics, type, field, coefficient, and the RMS errors of the
// residual (tabulated, orbits) and of the coefficient gradient (likewise).
#include <cstdio>
#include <cstring>
#include <random>

#include "p3_device.hpp"

using namespace femq;

typedef long double Ext;
using Tab = P3Basis<3, FEM_RULE_TET11>;
using Rule11 = RuleP2<3, FEM_RULE_TET11>;

template <int NC, typename Real>
static void ext_gradients(const Real* ij, const Real* u, Ext (&G)[11][NC][3]) {
    for (int q = 0; q < 11; ++q)
        for (int c = 0; c < NC; ++c) {
            Ext U[4] = {0, 0, 0, 0};
            for (int v = 0; v < 4; ++v)
                for (int b = 0; b < 20; ++b) U[v] += (Ext)Tab::dl(q, b, v) * u[b * NC + c];
            for (int i = 0; i < 3; ++i) G[q][c][i] = (U[1] - U[0]) * ij[i] + (U[2] - U[0]) * ij[3 + i] + (U[3] - U[0]) * ij[6 + i];
        }
}

// Residual r[20 * NC] and coefficient gradient dq[NM * 11] for w.
template <int NC, typename Real>
static void ext_element(const Real* ij, Real dj, const Real* u, const Real* w, const Real* aq, Ext* r, Ext* dq) {
    Ext G[11][NC][3], W[11][NC][3];
    ext_gradients<NC>(ij, u, G);
    ext_gradients<NC>(ij, w, W);
    for (int i = 0; i < 20 * NC; ++i) r[i] = 0;
    for (int q = 0; q < 11; ++q) {
        const Ext s = (Ext)Rule11::w(q) * std::fabs((Ext)dj);
        Ext f[NC][3], tu = 0, tw = 0, x = 0;
        for (int c = 0; c < NC; ++c) {
            tu += G[q][c][c];
            tw += W[q][c][c];
            for (int i = 0; i < 3; ++i) x += G[q][c][i] * (NC == 1 ? W[q][c][i] : W[q][c][i] + W[q][i % NC][c]);
        }
        dq[q] = s * (NC == 1 ? x : tu * tw);
        if (NC > 1) dq[11 + q] = s * x;
        for (int c = 0; c < NC; ++c) {
            for (int i = 0; i < 3; ++i)
                f[c][i] = NC == 1 ? aq[q] * G[q][c][i] : (Ext)aq[11 + q] * (G[q][c][i] + G[q][i % NC][c]) + (c == i ? aq[q] * tu : 0);
            Ext h[4] = {0, 0, 0, 0};
            for (int k = 0; k < 3; ++k) {
                for (int i = 0; i < 3; ++i) h[k + 1] += s * ij[k * 3 + i] * f[c][i];
                h[0] -= h[k + 1];
            }
            for (int b = 0; b < 20; ++b)
                for (int v = 0; v < 4; ++v) r[b * NC + c] += (Ext)Tab::dl(q, b, v) * h[v];
        }
    }
}

template <int PHYS, int NC, typename Real>
static void orbit_element(const Real* ij, Real dj, const Real* u, const Real* w, const Real* aq, Real* r, Real* dq) {
    constexpr int NM = NC == 1 ? 1 : 2;
    Real G[11][NC][3], W[11][NC][3];
    auto all = [&](const Real* x, Real(&g)[11][NC][3]) {
        for (int c = 0; c < NC; ++c)
            P3Tet::gradients<NC, Real>(x + c, ij, [&](auto q_c, const Real(&y)[3]) {
                for (int i = 0; i < 3; ++i) g[decltype(q_c)::value][c][i] = y[i];
            });
    };
    all(u, G);
    all(w, W);
    for (int q = 0; q < 11; ++q) {
        const Real s = Real(Rule11::w(q)) * fabs(dj);
        Real a[NM], tu = G[q][0][0], tw = W[q][0][0], x = Real(0);
        for (int c = 0; c < NC; ++c) {
            if (c > 0) { tu += G[q][c][c]; tw += W[q][c][c]; }
            for (int i = 0; i < 3; ++i) x = fmadd(G[q][c][i], NC == 1 ? W[q][c][i] : W[q][c][i] + W[q][i % NC][c], x);
        }
        dq[q] = NC == 1 ? x * s : tu * (s * tw);
        if (NC > 1) dq[11 + q] = x * s;
        for (int m = 0; m < NM; ++m) a[m] = s * aq[m * 11 + q];
        p3_weighted_flux<PHYS, NC, Real>(G[q], a);
    }
    for (int c = 0; c < NC; ++c) {
        Real x[20];
        P3Tet::scatter<Real>(ij, [&](auto q_c, int i) { return G[decltype(q_c)::value][c][i]; }, x);
        for (int b = 0; b < 20; ++b) r[b * NC + c] = x[b];
    }
}

// Barycentric coordinate v of node b.
static double node(int b, int v) {
    if (b < 4) return v == b;
    if (b >= 16) return v == 19 - b ? 0.0 : 1.0 / 3.0;
    using E = ElemP2<3, 0, 0, 0>;
    const int k = (b - 4) / 2, near = (b - 4) % 2 ? E::ej(k) : E::ei(k), far = (b - 4) % 2 ? E::ei(k) : E::ej(k);
    return v == near ? 2.0 / 3.0 : v == far ? 1.0 / 3.0 : 0.0;
}

template <int PHYS, typename Real>
static void measure(const char* name, int samples) {
    constexpr int NC = PHYS == FEM_ELASTICITY ? 3 : 1, NM = NC == 1 ? 1 : 2;
    const char* fields[] = {"independent", "offset", "linear", "smooth"};
    const char* coefs[] = {"independent", "constant", "spike"};
    for (int F = 0; F < 4; ++F)
        for (int C = 0; C < 3; ++C) {
            std::mt19937_64 gen(7 + F);
            auto U = [&] { return (double)(gen() >> 11) * 0x1p-53; };
            double e[4] = {0, 0, 0, 0};
            for (int t = 0; t < samples; ++t) {
                // a tetrahedron of the Kuhn cube, its vertices moved; every other one as it is
                static const int kuhn[4][3] = {{0, 0, 0}, {1, 0, 0}, {1, 1, 0}, {1, 1, 1}};
                const double h = 0.05, o[3] = {U(), U(), U()};
                double X[4][3], J[3][3], K[3][3];
                for (int v = 0; v < 4; ++v)
                    for (int i = 0; i < 3; ++i) X[v][i] = o[i] + h * (kuhn[v][i] + (t % 2) * 0.4 * (U() - 0.5));
                for (int i = 0; i < 3; ++i)
                    for (int k = 0; k < 3; ++k) J[i][k] = X[k + 1][i] - X[0][i];
                for (int i = 0; i < 3; ++i)
                    for (int k = 0; k < 3; ++k) {
                        const int a = (i + 1) % 3, b = (i + 2) % 3, c = (k + 1) % 3, d = (k + 2) % 3;
                        K[i][k] = J[a][c] * J[b][d] - J[a][d] * J[b][c];
                    }
                const double det = J[0][0] * K[0][0] + J[0][1] * K[0][1] + J[0][2] * K[0][2];
                Real ij[9], u[20 * NC], w[20 * NC], aq[11 * NM];
                for (int k = 0; k < 3; ++k)
                    for (int i = 0; i < 3; ++i) ij[k * 3 + i] = (Real)(K[i][k] / det);
                for (int b = 0; b < 20; ++b) {
                    double p[3] = {0, 0, 0};
                    for (int v = 0; v < 4; ++v)
                        for (int i = 0; i < 3; ++i) p[i] += node(b, v) * X[v][i];
                    for (int c = 0; c < NC; ++c) {
                        const double z = 2 * U() - 1, y = 2 * U() - 1;
                        const double s = std::sin(2 * p[0] + c) + std::cos(3 * p[1] - p[2] * c);
                        u[b * NC + c] = (Real)(F == 0 ? z : F == 1 ? 1000 + z : F == 2 ? (1 + c) * p[0] - p[2] + 0.3 : s);
                        w[b * NC + c] = (Real)(F == 0 ? y : F == 1 ? 100 + y : F == 2 ? p[1] + 0.5 : 0.5 * s + 0.1);
                    }
                }
                for (int i = 0; i < 11 * NM; ++i)
                    aq[i] = (Real)((0.5 + 1.5 * U()) * (C == 2 && i % 11 == t % 11 ? 1e4 : 1.0));
                if (C == 1)
                    for (int i = 0; i < 11 * NM; ++i) aq[i] = aq[i / 11 * 11];
                Ext R[20 * NC], D[11 * NM];
                Real r[2][20 * NC], d[2][11 * NM];
                ext_element<NC>(ij, (Real)det, u, w, aq, R, D);
                element_residual_p3<3, PHYS, FEM_RULE_TET11, Real>(ij, (Real)det, u, aq, r[0]);
                element_dcoef_points_p3<3, PHYS, FEM_RULE_TET11, Real>(ij, (Real)det, u, w, d[0]);
                orbit_element<PHYS, NC, Real>(ij, (Real)det, u, w, aq, r[1], d[1]);
                for (int k = 0; k < 2; ++k) {
                    for (int i = 0; i < 20 * NC; ++i) e[k] += (double)((r[k][i] - R[i]) * (r[k][i] - R[i]));
                    for (int i = 0; i < 11 * NM; ++i) e[2 + k] += (double)((d[k][i] - D[i]) * (d[k][i] - D[i]));
                }
            }
            std::printf("%s %s %s %s %.6e %.6e %.6e %.6e\n", name, sizeof(Real) == 4 ? "f32" : "f64", fields[F], coefs[C],
                        std::sqrt(e[0]), std::sqrt(e[1]), std::sqrt(e[2]), std::sqrt(e[3]));
        }
}

int main() {
    const int samples = 3000;
    measure<FEM_LAPLACE, float>("laplace", samples);
    measure<FEM_ELASTICITY, float>("elasticity", samples);
    measure<FEM_LAPLACE, double>("laplace", samples);
    measure<FEM_ELASTICITY, double>("elasticity", samples);
    return 0;
}
