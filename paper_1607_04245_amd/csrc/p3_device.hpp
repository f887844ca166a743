// p3_device.hpp -- element arithmetic of third-order (P3) Lagrange elements
// on affine simplices: the quadrature and basis phases of Eq. (2) with the
// P3 basis tabulated at the points (Section 3's B and D), one lane per
// element.
//
// Basis (node order: vertices v = 0..d; per edge (i, j), i < j,
// lexicographic, the node at 2/3 of lam_i then the node at 2/3 of lam_j; per
// face (i, j, k), lexicographic, its centroid):
//   vertex  lam_v (3 lam_v - 1)(3 lam_v - 2) / 2,
//   edge    (9/2) lam_a lam_o (3 lam_a - 1)   (a the nearer vertex),
//   face    27 lam_i lam_j lam_k.
// Each function's derivatives with respect to the barycentric coordinates
// at a quadrature point are compile-time constants (the points are), so a
// physical gradient is sum_v dphi/dlam_v g_v with g_v the gradients of the
// barycentric coordinates, and the tabulation costs no memory traffic: the
// quadrature phase forms U_v = sum_b dphi_b/dlam_v u_b (zero entries
// dropped at compile time), grad u = sum_v U_v g_v, and the basis phase
// adds dphi_b/dlam_v (g_v . w_q |J| f1) to every r_b. The rules are the
// degree-4 rules of the P2 path, which integrate a P3 stiffness entry with
// a constant coefficient exactly.
#pragma once

#include "p2_device.hpp"

namespace femq {

template <int DIM, int PHYS, int RULE, int SPACE>
struct ElemP3 {
    static constexpr int NV = DIM + 1;                              // vertices
    static constexpr int NE = DIM == 2 ? 3 : 6;                     // edges, two nodes each
    static constexpr int NF = DIM == 2 ? 1 : 4;                     // faces, one node each
    static constexpr int NB = NV + 2 * NE + NF;                     // 10 or 20
    static constexpr int NC = (PHYS == FEM_ELASTICITY) ? DIM : 1;
    static constexpr int NBT = NB * NC;
    static constexpr int NQ = RuleP2<DIM, RULE>::NQ;
    static constexpr int NW = SPACE == FEM_COEF_QUAD ? NQ : SPACE == FEM_COEF_P1 ? NV : 1;
    static constexpr int NCOEF = (PHYS == FEM_ELASTICITY) ? 2 : 1;
    static constexpr int NCQ = NCOEF * NW;
    static constexpr int NG = DIM * DIM;
};

// The P3 basis and its barycentric derivatives at point q of RULE.
template <int DIM, int RULE>
struct P3Basis {
    using Q = RuleP2<DIM, RULE>;
    static constexpr int NV = DIM + 1, NE = DIM == 2 ? 3 : 6;
    // edge k = (ei(k), ej(k)) and face f = (fa, fb, fc), lexicographic
    __host__ __device__ static constexpr int ei(int k) { return ElemP2<DIM, 0, RULE, 0>::ei(k); }
    __host__ __device__ static constexpr int ej(int k) { return ElemP2<DIM, 0, RULE, 0>::ej(k); }
    __host__ __device__ static constexpr int fa(int f) { return DIM == 2 ? 0 : (f < 3 ? 0 : 1); }
    __host__ __device__ static constexpr int fb(int f) { return DIM == 2 ? 1 : (f < 2 ? 1 : 2); }
    __host__ __device__ static constexpr int fc(int f) { return DIM == 2 ? 2 : (f == 0 ? 2 : 3); }

    __host__ __device__ static constexpr double phi(int q, int b) {
        if (b < NV) {
            const double l = Q::lam(q, b);
            return 0.5 * l * (3.0 * l - 1.0) * (3.0 * l - 2.0);
        }
        if (b < NV + 2 * NE) {
            const int k = (b - NV) / 2, s = (b - NV) % 2;
            const int a = s == 0 ? ei(k) : ej(k), o = s == 0 ? ej(k) : ei(k);
            return 4.5 * Q::lam(q, a) * Q::lam(q, o) * (3.0 * Q::lam(q, a) - 1.0);
        }
        const int f = b - NV - 2 * NE;
        return 27.0 * Q::lam(q, fa(f)) * Q::lam(q, fb(f)) * Q::lam(q, fc(f));
    }

    // d phi_b / d lam_v at point q
    __host__ __device__ static constexpr double dl(int q, int b, int v) {
        if (b < NV) {
            const double l = Q::lam(q, b);
            return v == b ? 0.5 * (27.0 * l * l - 18.0 * l + 2.0) : 0.0;
        }
        if (b < NV + 2 * NE) {
            const int k = (b - NV) / 2, s = (b - NV) % 2;
            const int a = s == 0 ? ei(k) : ej(k), o = s == 0 ? ej(k) : ei(k);
            const double la = Q::lam(q, a), lo = Q::lam(q, o);
            return v == a ? 4.5 * lo * (6.0 * la - 1.0) : (v == o ? 4.5 * la * (3.0 * la - 1.0) : 0.0);
        }
        const int f = b - NV - 2 * NE;
        const int i = fa(f), j = fb(f), k = fc(f);
        const double li = Q::lam(q, i), lj = Q::lam(q, j), lk = Q::lam(q, k);
        return v == i ? 27.0 * lj * lk : (v == j ? 27.0 * li * lk : (v == k ? 27.0 * li * lj : 0.0));
    }
};

// The basis values and barycentric derivatives at the points as a table,
// for lookups with a run-time (wave-uniform) function index.
template <int DIM, int RULE>
struct P3Table {
    static constexpr int NQ = RuleP2<DIM, RULE>::NQ, NB = ElemP3<DIM, 0, RULE, 0>::NB, NV = DIM + 1;
    double phi[NQ][NB];
    double dl[NQ][NB][NV];
    constexpr P3Table() : phi(), dl() {
        for (int q = 0; q < NQ; ++q)
            for (int b = 0; b < NB; ++b) {
                phi[q][b] = P3Basis<DIM, RULE>::phi(q, b);
                for (int v = 0; v < NV; ++v) dl[q][b][v] = P3Basis<DIM, RULE>::dl(q, b, v);
            }
    }
};

// Calls f(std::integral_constant<int, i>) for i = B .. E-1, so the basis
// values at a point are constant expressions: zero entries drop out at
// compile time and no loop is left to the optimizer's unrolling limits.
template <int B, int E, typename F>
__device__ __forceinline__ void unroll_for(const F& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>());
        unroll_for<B + 1, E>(f);
    }
}

// The P3 tetrahedron at the eleven-point rule. The points form three orbits
// (centroid; a high coordinate at one vertex; at both vertices of an edge), and as a
// function of the point du/dlam_v takes only a few shapes: its coefficients
// depend on lam_v and, at one other vertex p, on whether lam_p differs from
// the remaining two. The words of those two vertices share their coefficients,
// so they enter as pair sums, which serve every point: with
//   a_o = u(node near v on edge vo), b_o = u(node near o), f_o = u(face without o)
// a derivative takes u_v, the three pair sums and the three words of p, and at
// the centroid and at v's own vertex point u_v and the sums over all three: 77
// operations per v and component for all eleven points, where the products of
// the tabulated derivatives take 110. The basis phase is the transpose.
// Every word is multiplied by its own entry of the derivative table, as in the
// tabulated form, so nothing cancels that does not cancel there, and the terms
// are summed in orders that keep the partial sums small (small coefficients
// first, and a pair's next to the opposite ones). RMS rounding of the residual
// relative to the tabulated form's, both types: 0.73-0.93 over independent,
// constant plus independent, linear and smooth nodal fields, of dcoef 0.73-0.98.
// (Sums over all three vertices with the words of p as corrections take 53
// operations but cancel: 1.1-1.3 on linear and smooth fields.)
struct P3Tet {
    using Q = RuleP2<3, FEM_RULE_TET11>;
    // node of edge (v, o) near v; face without vertex p
    __host__ __device__ static constexpr int edge_node(int v, int o) {
        return 4 + 2 * ElemP2<3, 0, 0, 0>::edge_of(v, o) + (v < o ? 0 : 1);
    }
    __host__ __device__ static constexpr int face_without(int p) { return 19 - p; }
    // k-th vertex other than v
    __host__ __device__ static constexpr int other(int v, int k) { return k < v ? k : k + 1; }
    __host__ __device__ static constexpr int edge_point(int a, int b) { return 5 + ElemP2<3, 0, 0, 0>::edge_of(a, b); }
    // the edge that joins the two vertices other than a and b
    __host__ __device__ static constexpr int opposite_point(int a, int b) {
        return 5 + (5 - ElemP2<3, 0, 0, 0>::edge_of(a, b));
    }
    // The shapes of du/dlam_v: 0 centroid; 1 v's own vertex point; 2 another vertex
    // point (p high); 3 an edge point at v (p the other end); 4 an edge point
    // away from v (p the other low vertex).
    __host__ __device__ static constexpr int point(int k, int v, int p) {
        return k == 0 ? 0 : k == 1 ? 1 + v : k == 2 ? 1 + p : k == 3 ? edge_point(v, p) : opposite_point(v, p);
    }
    // Their coefficients, entries of the derivative table at v = 0 and p = 1: of
    // u_v (j = 0) and of a, b, f of the vertices that share one (j = 1..3),
    static constexpr double base(int k, int j) {
        return P3Basis<3, FEM_RULE_TET11>::dl(point(k, 0, 1), j == 0 ? 0 : j == 1 ? edge_node(0, 2) : j == 2 ? edge_node(2, 0)
                                                                                                    : face_without(3), 0);
    }
    // and of a, b, f of p (j = 1..3, shapes 2..4)
    static constexpr double own(int k, int j) {
        return P3Basis<3, FEM_RULE_TET11>::dl(point(k, 0, 1), j == 1 ? edge_node(0, 1) : j == 2 ? edge_node(1, 0) : face_without(1), 0);
    }
    // Order of the six terms after u_v in shapes 2..4: 1..3 the pair sums of a,
    // b, f, 4..6 p's own.
    static constexpr int term(int k, int i) {
        constexpr int order[3][6] = {{1, 6, 4, 3, 2, 5}, {5, 6, 2, 1, 3, 4}, {4, 5, 2, 1, 3, 6}};
        return order[k - 2][i];
    }

    // Physical gradient of one component at every point: u[b * NC] its words,
    // ij the inverse Jacobian; sink(q constant, gradient).
    template <int NC, typename Real, typename Sink>
    __device__ static __forceinline__ void gradients(const Real* u, const Real* ij, const Sink& sink) {
        Real d[11][4];
        unroll_for<0, 4>([&](auto v_c) {
            constexpr int v = decltype(v_c)::value;
            constexpr int o0 = other(v, 0), o1 = other(v, 1), o2 = other(v, 2);
            // x[j - 1]: a, b, f of the other vertices; y: their pair sums
            const Real x[3][3] = {{u[edge_node(v, o0) * NC], u[edge_node(v, o1) * NC], u[edge_node(v, o2) * NC]},
                                  {u[edge_node(o0, v) * NC], u[edge_node(o1, v) * NC], u[edge_node(o2, v) * NC]},
                                  {u[face_without(o0) * NC], u[face_without(o1) * NC], u[face_without(o2) * NC]}};
            Real y[3][3], z[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                y[j][0] = x[j][1] + x[j][2];
                y[j][1] = x[j][2] + x[j][0];
                y[j][2] = x[j][0] + x[j][1];
                z[j] = y[j][0] + x[j][0];
            }
            constexpr double c0 = base(0, 0), c1 = base(0, 1), c2 = base(0, 2), c3 = base(0, 3);
            d[0][v] = fmadd(Real(c3), z[2], fmadd(Real(c1), z[0], fmadd(Real(c2), z[1], Real(c0) * u[v * NC])));
            constexpr double v0 = base(1, 0), v1 = base(1, 1), v2 = base(1, 2), v3 = base(1, 3);
            d[1 + v][v] = fmadd(Real(v0), u[v * NC], fmadd(Real(v1), z[0], fmadd(Real(v2), z[1], Real(v3) * z[2])));
            unroll_for<2, 5>([&](auto k_c) {
                constexpr int k = decltype(k_c)::value;
                constexpr double b0 = base(k, 0);
                const Real t = Real(b0) * u[v * NC];
                unroll_for<0, 3>([&](auto n_c) {
                    constexpr int n = decltype(n_c)::value;
                    Real s = t;
                    unroll_for<0, 6>([&](auto i_c) {
                        constexpr int j = term(k, decltype(i_c)::value);
                        constexpr double c = j < 4 ? base(k, j) : own(k, j - 3);
                        s = fmadd(Real(c), j < 4 ? y[(j - 1) % 3][n] : x[(j - 1) % 3][n], s);
                    });
                    d[point(k, v, other(v, n))][v] = s;
                });
            });
        });
        unroll_for<0, 11>([&](auto q_c) {
            constexpr int q = decltype(q_c)::value;
            Real g[3];
#pragma unroll
            for (int i = 0; i < 3; ++i)
                g[i] = fmadd(d[q][3], ij[6 + i],
                             fmadd(d[q][2], ij[3 + i], fmadd(d[q][1], ij[i], d[q][0] * -((ij[i] + ij[3 + i]) + ij[6 + i]))));
            sink(q_c, g);
        });
    }

    // The transpose: r[b] of one component from the weighted flux at every
    // point, flux(q constant, i).
    template <typename Real, typename Flux>
    __device__ static __forceinline__ void scatter(const Real* ij, const Flux& flux, Real (&r)[20]) {
        Real h[11][4];  // g_v . flux
        unroll_for<0, 11>([&](auto q_c) {
            constexpr int q = decltype(q_c)::value;
            const Real f0 = flux(q_c, 0), f1 = flux(q_c, 1), f2 = flux(q_c, 2);
#pragma unroll
            for (int k = 0; k < 3; ++k) h[q][k + 1] = fmadd(ij[k * 3 + 2], f2, fmadd(ij[k * 3 + 1], f1, ij[k * 3] * f0));
            h[q][0] = fmadd(-((ij[2] + ij[5]) + ij[8]), f2, fmadd(-((ij[1] + ij[4]) + ij[7]), f1, -((ij[0] + ij[3]) + ij[6]) * f0));
        });
        unroll_for<0, 4>([&](auto v_c) {
            constexpr int v = decltype(v_c)::value;
            // x[k - 2]: h at the shape's points, y: pair sums, z: the sum of all three
            Real x[3][3], y[3][3], z[3];
            unroll_for<0, 3>([&](auto k_c) {
                constexpr int k = decltype(k_c)::value;
                x[k][0] = h[point(k + 2, v, other(v, 0))][v];
                x[k][1] = h[point(k + 2, v, other(v, 1))][v];
                x[k][2] = h[point(k + 2, v, other(v, 2))][v];
                y[k][0] = x[k][1] + x[k][2];
                y[k][1] = x[k][2] + x[k][0];
                y[k][2] = x[k][0] + x[k][1];
                z[k] = y[k][0] + x[k][0];
            });
            constexpr double c0 = base(0, 0), c1 = base(1, 0), c2 = base(2, 0), c3 = base(3, 0), c4 = base(4, 0);
            r[v] = fmadd(Real(c1), h[1 + v][v], fmadd(Real(c3), z[1], fmadd(Real(c2), z[0], fmadd(Real(c4), z[2], Real(c0) * h[0][v]))));
            unroll_for<1, 4>([&](auto j_c) {
                constexpr int j = decltype(j_c)::value;
                constexpr double b0 = base(0, j), b1 = base(1, j), b2 = base(2, j), b3 = base(3, j), b4 = base(4, j);
                constexpr double w2 = own(2, j), w3 = own(3, j), w4 = own(4, j);
                const Real t = fmadd(Real(b0), h[0][v], Real(b1) * h[1 + v][v]);
                unroll_for<0, 3>([&](auto n_c) {
                    constexpr int n = decltype(n_c)::value, p = other(v, n);
                    constexpr int b = j == 1 ? edge_node(v, p) : j == 2 ? edge_node(p, v) : face_without(p);
                    // an edge node is met at both its vertices, a face at its three
                    constexpr bool first = j < 3 ? v < p : v == (p == 0 ? 1 : 0);
                    const Real s = fmadd(Real(b4), y[2][n], fmadd(Real(b3), y[1][n], fmadd(Real(b2), y[0][n], t)));
                    const Real e = fmadd(Real(w4), x[2][n], fmadd(Real(w3), x[1][n], fmadd(Real(w2), x[0][n], s)));
                    if constexpr (first) r[b] = e;
                    else r[b] += e;
                });
            });
        });
    }
};

// f1 of the forms with a gradient term at one point, in place, from
// coefficients that already carry the weight.
template <int PHYS, int NC, typename Real>
__device__ __forceinline__ void p3_weighted_flux(Real (&g)[NC][3], const Real* a) {
    if constexpr (PHYS == FEM_LAPLACE) {
#pragma unroll
        for (int i = 0; i < 3; ++i) g[0][i] *= a[0];
    } else {
        const Real lt = a[0] * ((g[0][0] + g[1][1]) + g[2][2]), m2 = a[1] + a[1];
        const Real s01 = a[1] * (g[0][1] + g[1][0]), s02 = a[1] * (g[0][2] + g[2][0]), s12 = a[1] * (g[1][2] + g[2][1]);
#pragma unroll
        for (int c = 0; c < 3; ++c) g[c][c] = fmadd(m2, g[c][c], lt);
        g[0][1] = g[1][0] = s01;
        g[0][2] = g[2][0] = s02;
        g[1][2] = g[2][1] = s12;
    }
}

// The coefficient words of element e turned into values at the points: the
// space is a uniform run-time branch (one kernel per dimension, physics and
// type), the arithmetic after it is the same for every space. STREAM: the
// loads bypass the caches' retention (each word is read once); kernels whose
// tiles share cache lines read through the caches.
template <int DIM, int PHYS, int RULE, typename Real, bool STREAM = true>
__device__ __forceinline__ void p3_coef_points(int space, const Real* __restrict__ coef, int64_t n, int64_t e,
                                               Real (&aq)[ElemP3<DIM, PHYS, RULE, FEM_COEF_QUAD>::NCQ]) {
    using E = ElemP3<DIM, PHYS, RULE, FEM_COEF_QUAD>;
    using Q = RuleP2<DIM, RULE>;
    auto load = [](const Real* p) {
        if constexpr (STREAM) return __builtin_nontemporal_load(p);
        else return *p;
    };
    if (space == FEM_COEF_QUAD) {
#pragma unroll
        for (int f = 0; f < E::NCQ; ++f) aq[f] = load(coef + f * n + e);
    } else if (space == FEM_COEF_P1) {
#pragma unroll
        for (int m = 0; m < E::NCOEF; ++m) {
            Real c[E::NV];
#pragma unroll
            for (int v = 0; v < E::NV; ++v) c[v] = load(coef + (m * E::NV + v) * n + e);
#pragma unroll
            for (int q = 0; q < E::NQ; ++q) {
                Real t = Real(Q::lam(q, 0)) * c[0];
#pragma unroll
                for (int v = 1; v < E::NV; ++v) t = fmadd(Real(Q::lam(q, v)), c[v], t);
                aq[m * E::NQ + q] = t;
            }
        }
    } else {
#pragma unroll
        for (int m = 0; m < E::NCOEF; ++m) {
            const Real c = load(coef + m * n + e);
#pragma unroll
            for (int q = 0; q < E::NQ; ++q) aq[m * E::NQ + q] = c;
        }
    }
}

// Residual of one P3 element: r[b*NC + c], from invJ ij[k*DIM + i], det J,
// closure u[b*NC + c] and the coefficient values at the points
// aq[m*NQ + q].
template <int DIM, int PHYS, int RULE, typename Real>
__device__ __forceinline__ void element_residual_p3(const Real* ij, Real dj, const Real* u, const Real* aq, Real* r) {
    using E = ElemP3<DIM, PHYS, RULE, FEM_COEF_QUAD>;
    using Q = RuleP2<DIM, RULE>;
    using T = P3Basis<DIM, RULE>;
    using P = Physics<PHYS>;
    constexpr int NC = E::NC, NV = E::NV, NB = E::NB;
#pragma unroll
    for (int b = 0; b < E::NBT; ++b) r[b] = Real(0);
    const Real adj = fabs(dj);
    Real g[NV][DIM];
    p2_bary_grads<DIM, Real>(ij, g);
    unroll_for<0, E::NQ>([&](auto q_c) {
        constexpr int q = decltype(q_c)::value;
        Real uq[NC], gq[NC][DIM];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if constexpr (P::NEEDS_U) {
                Real s = Real(0);
                unroll_for<0, NB>([&](auto b_c) {
                    constexpr int b = decltype(b_c)::value;
                    s = fmadd(Real(T::phi(q, b)), u[b * NC + c], s);
                });
                uq[c] = s;
            }
            if constexpr (P::HAS_F1) {
                Real U[NV];
                unroll_for<0, NV>([&](auto v_c) {
                    constexpr int v = decltype(v_c)::value;
                    Real s = Real(0);
                    unroll_for<0, NB>([&](auto b_c) {
                        constexpr int b = decltype(b_c)::value;
                        constexpr double d = T::dl(q, b, v);
                        if constexpr (d != 0.0) s = fmadd(Real(d), u[b * NC + c], s);
                    });
                    U[v] = s;
                });
#pragma unroll
                for (int i = 0; i < DIM; ++i) {
                    Real s = U[0] * g[0][i];
#pragma unroll
                    for (int v = 1; v < NV; ++v) s = fmadd(U[v], g[v][i], s);
                    gq[c][i] = s;
                }
            }
        }
        Real a[E::NCOEF];
#pragma unroll
        for (int m = 0; m < E::NCOEF; ++m) a[m] = aq[m * E::NQ + q];
        Real f0[NC], f1[NC][DIM];
        P::template point<DIM, Real>(uq, gq, a, f0, f1);
        const Real s = Real(Q::w(q)) * adj;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if constexpr (P::HAS_F1) {
                Real h[NV];  // g_v . (w_q |J| f1)
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    Real t = g[v][0] * f1[c][0];
#pragma unroll
                    for (int i = 1; i < DIM; ++i) t = fmadd(g[v][i], f1[c][i], t);
                    h[v] = s * t;
                }
                unroll_for<0, NB>([&](auto b_c) {
                    constexpr int b = decltype(b_c)::value;
                    unroll_for<0, NV>([&](auto v_c) {
                        constexpr int v = decltype(v_c)::value;
                        constexpr double d = T::dl(q, b, v);
                        if constexpr (d != 0.0) r[b * NC + c] = fmadd(Real(d), h[v], r[b * NC + c]);
                    });
                });
            }
            if constexpr (P::HAS_F0) {
                const Real sf = s * f0[c];
                unroll_for<0, NB>([&](auto b_c) {
                    constexpr int b = decltype(b_c)::value;
                    r[b * NC + c] = fmadd(Real(T::phi(q, b)), sf, r[b * NC + c]);
                });
            }
        }
    });
}

// Derivative of L = w . R with respect to the coefficient values at the
// points (the forms are linear in the coefficients): dq[m*NQ + q] =
// w_q |J| [w^q . f0(u; e_m) + grad w : f1(u; e_m)].
template <int DIM, int PHYS, int RULE, typename Real>
__device__ __forceinline__ void element_dcoef_points_p3(const Real* ij, Real dj, const Real* u, const Real* w,
                                                        Real* dq) {
    using E = ElemP3<DIM, PHYS, RULE, FEM_COEF_QUAD>;
    using Q = RuleP2<DIM, RULE>;
    using T = P3Basis<DIM, RULE>;
    using P = Physics<PHYS>;
    constexpr int NC = E::NC, NV = E::NV, NB = E::NB;
    const Real adj = fabs(dj);
    Real g[NV][DIM];
    p2_bary_grads<DIM, Real>(ij, g);
    // value and physical gradient of a field at point q
    auto field_at = [&](auto q_c, const Real* f, Real (&fq)[NC], Real (&gf)[NC][DIM]) {
        constexpr int q = decltype(q_c)::value;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if constexpr (P::HAS_F0) {
                Real s = Real(0);
                unroll_for<0, NB>([&](auto b_c) {
                    constexpr int b = decltype(b_c)::value;
                    s = fmadd(Real(T::phi(q, b)), f[b * NC + c], s);
                });
                fq[c] = s;
            }
            if constexpr (P::HAS_F1) {
                Real U[NV];
                unroll_for<0, NV>([&](auto v_c) {
                    constexpr int v = decltype(v_c)::value;
                    Real s = Real(0);
                    unroll_for<0, NB>([&](auto b_c) {
                        constexpr int b = decltype(b_c)::value;
                        constexpr double d = T::dl(q, b, v);
                        if constexpr (d != 0.0) s = fmadd(Real(d), f[b * NC + c], s);
                    });
                    U[v] = s;
                });
#pragma unroll
                for (int i = 0; i < DIM; ++i) {
                    Real s = U[0] * g[0][i];
#pragma unroll
                    for (int v = 1; v < NV; ++v) s = fmadd(U[v], g[v][i], s);
                    gf[c][i] = s;
                }
            }
        }
    };
    unroll_for<0, E::NQ>([&](auto q_c) {
        constexpr int q = decltype(q_c)::value;
        Real uq[NC], gu[NC][DIM], wq[NC], gw[NC][DIM];
        field_at(q_c, u, uq, gu);
        field_at(q_c, w, wq, gw);
        const Real s = Real(Q::w(q)) * adj;
#pragma unroll
        for (int m = 0; m < E::NCOEF; ++m) {
            Real a[E::NCOEF];
#pragma unroll
            for (int mm = 0; mm < E::NCOEF; ++mm) a[mm] = Real(mm == m ? 1 : 0);
            Real f0[NC], f1[NC][DIM];
            P::template point<DIM, Real>(uq, gu, a, f0, f1);
            Real acc = Real(0);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                if constexpr (P::HAS_F0) acc = fmadd(wq[c], f0[c], acc);
                if constexpr (P::HAS_F1) {
#pragma unroll
                    for (int i = 0; i < DIM; ++i) acc = fmadd(gw[c][i], f1[c][i], acc);
                }
            }
            dq[m * E::NQ + q] = s * acc;
        }
    });
}

}  // namespace femq
