// jacobian.hip -- element matrices K_e = dR_e / du_e of the forms of Eq. (1)
// for P1 and P2 Lagrange elements, from precomputed affine geometry.
//
// Differentiating the bracket of Eq. (2) with respect to the closure puts
// the pointwise derivatives of f0 and f1 between the basis values and
// physical gradients:
//   K[(b,c),(b',c')] = sum_q w_q |J| ( phi_b g0 phi_b'
//                      + sum_ij G_b,i g3[c][i][c'][j] G_b',j ),
// Laplacian g3 = kappa delta_ij, elasticity g3 = lambda delta_ci delta_c'j
// + mu (delta_cc' delta_ij + delta_cj delta_ic'), mass g0 = kappa.
//
// A lane owns V consecutive elements; every SoA row is one coalesced access per
// wave, and the output (N_bt^2 rows) dominates the traffic. The rule and coefficient
// space only enter the moments below, so they are uniform run-time
// arguments of one kernel per (dim, physics, order, dtype). The gradient terms use the
// barycentric structure of the basis: grad phi_b = sum_v alpha_bv grad lam_v
// with alpha_bv affine in the barycentric coordinates (P1: alpha = delta;
// P2 vertex v: 4 lam_v - 1; P2 edge (i, j): 4 lam_j at i and 4 lam_i at j).
// The quadrature sum then reduces to weighted moments of the coefficient,
//   m0 = sum_q k_q, m1_v = sum_q k_q lam_v, m2_vw = sum_q k_q lam_v lam_w,
// k_q = w_q |J| a(x_q), computed once per element, and each matrix entry is
// a short combination of moments and the products g_v . g_w of the physical
// barycentric gradients. The mass term (products of basis values) is summed
// over the points directly. The matrix is written exactly symmetric: each
// entry below the diagonal is a copy of its mirror. On small meshes blockIdx.y
// deals the basis functions out to several workgroups per tile (matrix_parts).
#include "fem_device.hpp"
#include "fem_internal.hpp"
#include "p2_device.hpp"

namespace femq {

// Quadrature rules of both orders as barycentric points: the degree-2 and
// degree-4 rules, and the one-point centroid rule.
template <int DIM, int RULE>
struct RuleBary : RuleP2<DIM, RULE> {};

template <int DIM>
struct RuleBary<DIM, FEM_RULE_CENTROID> {
    static constexpr int NQ = 1;
    __host__ __device__ static constexpr double lam(int, int) { return 1.0 / (DIM + 1); }
    __host__ __device__ static constexpr double w(int) { return DIM == 2 ? 0.5 : 1.0 / 6.0; }
};

// alpha = a0 + a1 * lam_u (u < 0: constant)
struct Aff {
    double a0;
    int u;
    double a1;
};

// Lagrange basis of order 1 or 2; node order: vertices, then edges (i, j),
// i < j, lexicographic.
template <int DIM, int ORDER>
struct LagBasis {
    static constexpr int NV = DIM + 1;
    static constexpr int NE = DIM == 2 ? 3 : 6;
    static constexpr int NB = ORDER == 1 ? NV : NV + NE;
    __host__ __device__ static constexpr int ei(int k) {
        return DIM == 2 ? (k < 2 ? 0 : 1) : (k < 3 ? 0 : (k < 5 ? 1 : 2));
    }
    __host__ __device__ static constexpr int ej(int k) {
        return DIM == 2 ? (k < 2 ? k + 1 : 2) : (k < 3 ? k + 1 : (k < 5 ? k - 1 : 3));
    }
    // barycentric gradients in grad phi_b: one (vertex functions) or two (edges)
    __host__ __device__ static constexpr int nsupp(int b) { return (ORDER == 1 || b < NV) ? 1 : 2; }
    __host__ __device__ static constexpr int supp(int b, int s) {
        return (ORDER == 1 || b < NV) ? b : (s == 0 ? ei(b - NV) : ej(b - NV));
    }
    __host__ __device__ static constexpr Aff alpha(int b, int s) {
        return ORDER == 1 ? Aff{1.0, -1, 0.0}
             : b < NV     ? Aff{-1.0, b, 4.0}
             : s == 0     ? Aff{0.0, ej(b - NV), 4.0}
                          : Aff{0.0, ei(b - NV), 4.0};
    }
    // phi_b at a point with barycentric coordinates lam(v)
    template <typename L>
    __host__ __device__ static constexpr double value(int b, const L& lam) {
        return ORDER == 1 ? lam(b)
             : b < NV     ? lam(b) * (2.0 * lam(b) - 1.0)
                          : 4.0 * lam(ei(b - NV)) * lam(ej(b - NV));
    }
};

// Calls f(std::integral_constant<int, i>) for i = B .. E-1: loops whose
// bounds depend on an outer index stay compile-time constants.
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(const F& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>());
        static_for<B + 1, E>(f);
    }
}

template <int NV, typename Real>
struct Moments {
    Real m0;
    Real m1[NV];
    Real m2[NV][NV];
};

// sum_q k_q alpha_A(q) alpha_B(q) from the moments; constant factors fold at
// compile time once the callers' loops are unrolled.
template <int NV, typename Real>
__device__ __forceinline__ Real moment(const Moments<NV, Real>& M, Aff A, Aff B) {
    const int ua = A.u < 0 ? 0 : A.u, ub = B.u < 0 ? 0 : B.u;
    Real s = Real(0);
    if (A.a0 != 0.0 && B.a0 != 0.0) s = Real(A.a0 * B.a0) * M.m0;
    if (A.a0 != 0.0 && B.a1 != 0.0) s = fmadd(Real(A.a0 * B.a1), M.m1[ub], s);
    if (A.a1 != 0.0 && B.a0 != 0.0) s = fmadd(Real(A.a1 * B.a0), M.m1[ua], s);
    if (A.a1 != 0.0 && B.a1 != 0.0) s = fmadd(Real(A.a1 * B.a1), M.m2[ua][ub], s);
    return s;
}

// Coefficient words of a space.
template <int DIM, int RULE, int SPACE>
constexpr int coef_words() {
    return SPACE == FEM_COEF_QUAD ? RuleBary<DIM, RULE>::NQ : SPACE == FEM_COEF_P1 ? DIM + 1 : 1;
}

// Coefficient at the points of the rule, weighted: k[m][q] = w_q |J| a_m(x_q)
// from the words cf[][v] of the lane's element v in their space.
template <int DIM, int RULE, int SPACE, int NCOEF, int W, typename Real>
__device__ __forceinline__ void weighted_coef(const Real (&cf)[NCOEF * coef_words<DIM, RULE, SPACE>()][W], int v, Real dj,
                                              Real (&k)[NCOEF][RuleBary<DIM, RULE>::NQ]) {
    using Q = RuleBary<DIM, RULE>;
    constexpr int NV = DIM + 1, NQ = Q::NQ, NW = coef_words<DIM, RULE, SPACE>();
#pragma unroll
    for (int m = 0; m < NCOEF; ++m) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            Real a;
            if constexpr (SPACE == FEM_COEF_QUAD) {
                a = cf[m * NW + q][v];
            } else if constexpr (SPACE == FEM_COEF_P1) {
                a = Real(Q::lam(q, 0)) * cf[m * NW][v];
#pragma unroll
                for (int w = 1; w < NV; ++w) a = fmadd(Real(Q::lam(q, w)), cf[m * NW + w][v], a);
            } else {
                a = cf[m * NW][v];
            }
            k[m][q] = (Real(Q::w(q)) * dj) * a;
        }
    }
}

// Moments of the weighted coefficients (m1, m2 only for second order).
template <int DIM, int RULE, int SPACE, int NCOEF, int ORDER, int W, typename Real>
__device__ __forceinline__ void coef_moments(const Real (&cf)[NCOEF * coef_words<DIM, RULE, SPACE>()][W], int lane_elem,
                                             Real dj, Moments<DIM + 1, Real> (&M)[NCOEF]) {
    using Q = RuleBary<DIM, RULE>;
    constexpr int NV = DIM + 1, NQ = Q::NQ;
    Real k[NCOEF][NQ];
    weighted_coef<DIM, RULE, SPACE, NCOEF, W, Real>(cf, lane_elem, dj, k);
#pragma unroll
    for (int m = 0; m < NCOEF; ++m) {
        Real s = k[m][0];
#pragma unroll
        for (int q = 1; q < NQ; ++q) s += k[m][q];
        M[m].m0 = s;
        if constexpr (ORDER == 2) {
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                Real s1 = Real(0);
#pragma unroll
                for (int q = 0; q < NQ; ++q) s1 = fmadd(Real(Q::lam(q, v)), k[m][q], s1);
                M[m].m1[v] = s1;
#pragma unroll
                for (int w = 0; w < NV; ++w) {
                    if (w < v) continue;
                    Real s2 = Real(0);
#pragma unroll
                    for (int q = 0; q < NQ; ++q) s2 = fmadd(Real(Q::lam(q, v) * Q::lam(q, w)), k[m][q], s2);
                    M[m].m2[v][w] = s2;
                    M[m].m2[w][v] = s2;
                }
            }
        }
    }
}

// Words e .. e+W-1 of entry (r, s) of a matrix with `size` rows, and of its
// mirror.
template <bool STREAM_OUT, typename Real, int W>
__device__ __forceinline__ void store_entry(const Real (&x)[1][W], int r, int s, int size, Real* __restrict__ out, int64_t n,
                                            int64_t e) {
    store_rows_v<1, STREAM_OUT>(out + (int64_t)(r * size + s) * n, n, e, x);
    if (s != r) store_rows_v<1, STREAM_OUT>(out + (int64_t)(s * size + r) * n, n, e, x);
}

// Mass matrix K_bb' = sum_q k_q phi_b(x_q) phi_b'(x_q), stored directly.
template <int DIM, int ORDER, int RULE, int SPACE, bool STREAM_OUT, bool SPLIT, int W, typename Real>
__device__ __forceinline__ void mass_matrix(const Real* __restrict__ coef, int64_t n, int64_t e, const Real (&dj)[1][W],
                                            Real* __restrict__ out) {
    using Q = RuleBary<DIM, RULE>;
    using Bs = LagBasis<DIM, ORDER>;
    constexpr int NB = Bs::NB, NQ = Q::NQ, NW = coef_words<DIM, RULE, SPACE>();
    Real cf[NW][W], k[W][1][NQ];
    load_rows_v<NW>(coef, n, e, cf);
#pragma unroll
    for (int v = 0; v < W; ++v) weighted_coef<DIM, RULE, SPACE, 1, W, Real>(cf, v, fabs(dj[0][v]), k[v]);
    static_for<0, NB>([&](auto b_c) {
        constexpr int b = decltype(b_c)::value;
        if (SPLIT && b % gridDim.y != blockIdx.y) return;
        static_for<b, NB>([&](auto bp_c) {
            constexpr int bp = decltype(bp_c)::value;
            Real x[1][W];
#pragma unroll
            for (int v = 0; v < W; ++v) {
                Real s = Real(0);
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    auto lam = [q](int w) { return Q::lam(q, w); };
                    s = fmadd(Real(Bs::value(b, lam) * Bs::value(bp, lam)), k[v][0][q], s);
                }
                x[0][v] = s;
            }
            store_entry<STREAM_OUT>(x, b, bp, NB, out, n, e);
        });
    });
}

// Calls f(rule constant, space constant) for the element's (rule, space):
// order 1 takes the degree-2 rule or the centroid, order 2 the degree-2 or
// the degree-4 rule. The host validates the pair; the arguments are uniform
// over the grid, so the branch is scalar. With one point, point values and a
// constant are the same words and the same code, so they take one branch: of two
// branches alike the compiler kept one and lost the other's |J| on its way there (P1
// mass matrices, kernels that deal out no basis functions).
template <int DIM, int ORDER, typename F>
__device__ __forceinline__ void with_scheme(int rule, int space, const F& f) {
    constexpr int LOW = DIM == 2 ? FEM_RULE_TRI3 : FEM_RULE_TET4;
    constexpr int OTHER = ORDER == 1 ? FEM_RULE_CENTROID : (DIM == 2 ? FEM_RULE_TRI6 : FEM_RULE_TET11);
    auto by_space = [&](auto rule_c) {
        constexpr bool one_point = RuleBary<DIM, decltype(rule_c)::value>::NQ == 1;
        if (!one_point && space == FEM_COEF_QUAD) f(rule_c, std::integral_constant<int, FEM_COEF_QUAD>());
        else if (space == FEM_COEF_P1) f(rule_c, std::integral_constant<int, FEM_COEF_P1>());
        else f(rule_c, std::integral_constant<int, FEM_COEF_P0>());
    };
    if (rule == LOW) by_space(std::integral_constant<int, LOW>());
    else by_space(std::integral_constant<int, OTHER>());
}

// Matrix entries between basis functions b and bp of one element, from its
// moments, gradients and their products.
template <int DIM, int PHYS, int ORDER, int b, int bp, int NC, int NCOEF, typename Real>
__device__ __forceinline__ void matrix_block(const Moments<DIM + 1, Real> (&M)[NCOEF], const Real (&g)[DIM + 1][DIM],
                                             const Real (&P)[DIM + 1][DIM + 1], Real (&blk)[NC][NC]) {
    using Bs = LagBasis<DIM, ORDER>;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int cp = 0; cp < NC; ++cp) blk[c][cp] = Real(0);
#pragma unroll
    for (int s = 0; s < Bs::nsupp(b); ++s)
#pragma unroll
        for (int t = 0; t < Bs::nsupp(bp); ++t) {
            const int v = Bs::supp(b, s), w = Bs::supp(bp, t);
            const Aff A = Bs::alpha(b, s), B = Bs::alpha(bp, t);
            if constexpr (PHYS == FEM_LAPLACE) {
                blk[0][0] = fmadd(moment(M[0], A, B), P[v][w], blk[0][0]);
            } else {
                const Real lm = moment(M[0], A, B), mu = moment(M[1], A, B);
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int cp = 0; cp < NC; ++cp) {
                        if (bp == b && cp < c) continue;
                        Real x = fmadd(lm * g[v][c], g[w][cp], blk[c][cp]);
                        x = fmadd(mu, g[v][cp] * g[w][c], x);
                        if (c == cp) x = fmadd(mu, P[v][w], x);
                        blk[c][cp] = x;
                    }
            }
        }
}

// SPLIT: blockIdx.y deals out the basis functions. The test of it also keeps
// one function's arithmetic and stores apart from the next one's. Short rows
// lose by that, so launches that need no split go without (P2 3D Laplacian
// FP64, 262,144 tets: 53.0 us with it, 49.9 without); the elasticity blocks of
// V elements need it (3D FP32, V = 4: 133 registers with it, 271 without,
// 400,000 tets 54 and 61 us).
template <int DIM, int PHYS, int ORDER, int V, bool STREAM_OUT, bool SPLIT, typename Real>
__global__ void __launch_bounds__(256)
jacobian_kernel(int64_t n, int order, int rule, int space, const Real* __restrict__ inv_j, const Real* __restrict__ det_j,
                const Real* __restrict__ coef, Real* __restrict__ out) {
    using Bs = LagBasis<DIM, ORDER>;
    constexpr int NV = DIM + 1, NB = Bs::NB;
    constexpr int NC = PHYS == FEM_ELASTICITY ? DIM : 1, NBT = NB * NC;
    constexpr int NCOEF = PHYS == FEM_ELASTICITY ? 2 : 1;
    const int64_t nchunk = (n + V - 1) / V;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t ch = (V == 1 ? row_block<STREAM_OUT>(order) : row_block(order)) * blockDim.x + threadIdx.x; ch < nchunk; ch += stride) {
        for_chunk<V>(ch * V, n, [&](auto width, int64_t e) {
            constexpr int W = decltype(width)::value;
            Real dj[1][W];
            load_rows_v<1>(det_j, n, e, dj);
            if constexpr (PHYS == FEM_MASS) {
                with_scheme<DIM, ORDER>(rule, space, [&](auto rule_c, auto space_c) {
                    mass_matrix<DIM, ORDER, decltype(rule_c)::value, decltype(space_c)::value, STREAM_OUT, SPLIT, W, Real>(
                        coef, n, e, dj, out);
                });
            } else {
                Moments<NV, Real> M[W][NCOEF];
                with_scheme<DIM, ORDER>(rule, space, [&](auto rule_c, auto space_c) {
                    constexpr int R = decltype(rule_c)::value, S = decltype(space_c)::value;
                    Real cf[NCOEF * coef_words<DIM, R, S>()][W];
                    load_rows_v<NCOEF * coef_words<DIM, R, S>()>(coef, n, e, cf);
#pragma unroll
                    for (int v = 0; v < W; ++v)
                        coef_moments<DIM, R, S, NCOEF, ORDER, W, Real>(cf, v, fabs(dj[0][v]), M[v]);
                });
                Real ij[DIM * DIM][W];
                load_rows_v<DIM * DIM>(inv_j, n, e, ij);
                Real g[W][NV][DIM];  // physical barycentric gradients: g_{k+1} = row k of J^{-1}, g_0 = -sum
                Real P[W][NV][NV];   // g_v . g_w
#pragma unroll
                for (int x = 0; x < W; ++x) {
#pragma unroll
                    for (int i = 0; i < DIM; ++i) {
                        Real s = Real(0);
#pragma unroll
                        for (int kk = 0; kk < DIM; ++kk) {
                            g[x][kk + 1][i] = ij[kk * DIM + i][x];
                            s += ij[kk * DIM + i][x];
                        }
                        g[x][0][i] = -s;
                    }
#pragma unroll
                    for (int v = 0; v < NV; ++v)
#pragma unroll
                        for (int w = 0; w < NV; ++w) {
                            if (w < v) continue;
                            Real s = g[x][v][0] * g[x][w][0];
#pragma unroll
                            for (int i = 1; i < DIM; ++i) s = fmadd(g[x][v][i], g[x][w][i], s);
                            P[x][v][w] = s;
                            P[x][w][v] = s;
                        }
                }
                static_for<0, NB>([&](auto b_c) {
                    constexpr int b = decltype(b_c)::value;
                    if (SPLIT && b % gridDim.y != blockIdx.y) return;
                    static_for<b, NB>([&](auto bp_c) {
                        constexpr int bp = decltype(bp_c)::value;
                        Real blk[W][NC][NC];
#pragma unroll
                        for (int x = 0; x < W; ++x)
                            matrix_block<DIM, PHYS, ORDER, b, bp, NC, NCOEF, Real>(M[x], g[x], P[x], blk[x]);
#pragma unroll
                        for (int c = 0; c < NC; ++c)
#pragma unroll
                            for (int cp = 0; cp < NC; ++cp) {
                                if (bp == b && cp < c) continue;
                                Real x[1][W];
#pragma unroll
                                for (int v = 0; v < W; ++v) x[0][v] = blk[v][c][cp];
                                store_entry<STREAM_OUT>(x, b * NC + c, bp * NC + cp, NBT, out, n, e);
                            }
                    });
                });
            }
        });
    }
}

// Elements per lane, V: 16 bytes of every row for P1, where the matrices are
// short enough for V sets of moments and gradients in the registers.
//  - Elasticity, as long as that leaves a wave per SIMD, in FP32 at odd words two.
//    Odd words, four waves per workgroup: 3D FP32, 327,691 tets 63 us with V = 1,
//    69 with 4, 524,309 tets 101 and 80; FP64, 163,859 tets 57 and 56, 2^20 + 3 tets
//    354 and 342. Whole lines: 3D FP32, 327,680 tets 50 and 46; FP64, 400,000 tets
//    112 and 107 (518 MB, 4.8 TB/s).
//  - Laplacian and mass FP32 at odd words, as long as that leaves two: 3D,
//    1,000,001 tets 26.8 and 24.4 us, mass 20.4 and 18.3; but 300,001 tets 9.2
//    and 11.2. Whole lines lose (FP64, 2^20 tets 46 and 52), FP64 at odd words
//    is the same.
template <int DIM, int PHYS, int ORDER, typename Real>
static hipError_t launch_jac(int rule, int space, const JacobianArgs& a, const Launch& l) {
    constexpr bool ELAST = PHYS == FEM_ELASTICITY;
    constexpr int V = ORDER == 1 && (ELAST || sizeof(Real) == 4) ? 16 / (int)sizeof(Real) : 1;
    Launch m = l;
    auto go = [&](auto k, int parts) {
        hipLaunchKernelGGL(k, dim3(m.grid, parts), dim3(m.block), 0, m.stream, a.n, m.order, rule, space,
                           static_cast<const Real*>(a.inv_j), static_cast<const Real*>(a.det_j),
                           static_cast<const Real*>(a.coef), static_cast<Real*>(a.out));
        return hipGetLastError();
    };
    if constexpr (V > 1) {
        const int64_t waves = ELAST && (l.stream_out || sizeof(Real) == 8) ? 1024 : 2048;
        if (a.n >= V * 64 * waves && (ELAST || !l.stream_out)) {
            m.grid = grid_for_lanes(l, (a.n + V - 1) / V);
            if constexpr (ELAST) {
                if (l.stream_out) return go(jacobian_kernel<DIM, PHYS, ORDER, V, true, true, Real>, 1);
            }
            return go(jacobian_kernel<DIM, PHYS, ORDER, V, false, ELAST, Real>, 1);
        }
    }
    const int parts = matrix_parts(l, a.n, LagBasis<DIM, ORDER>::NB, kMatrixWaves);
    if (parts > 1) return l.stream_out ? go(jacobian_kernel<DIM, PHYS, ORDER, 1, true, true, Real>, parts)
                                       : go(jacobian_kernel<DIM, PHYS, ORDER, 1, false, true, Real>, parts);
    return l.stream_out ? go(jacobian_kernel<DIM, PHYS, ORDER, 1, true, false, Real>, 1)
                        : go(jacobian_kernel<DIM, PHYS, ORDER, 1, false, false, Real>, 1);
}

// Runtime (dim, physics, order, dtype) to a kernel instance; (rule, space)
// are kernel arguments. Rules: order 1 takes the degree-2 rule of its
// dimension or the centroid, order 2 the degree-2 or the degree-4 rule.
hipError_t launch_jacobian(int dim, int phys, int order, int rule, int space, int dtype, const JacobianArgs& a,
                           const Launch& l) {
    const int low = dim == 2 ? FEM_RULE_TRI3 : FEM_RULE_TET4, high = dim == 2 ? FEM_RULE_TRI6 : FEM_RULE_TET11;
    const bool rule_ok = rule == low || (order == 1 && rule == FEM_RULE_CENTROID) || (order == 2 && rule == high);
    const bool space_ok = space == FEM_COEF_QUAD || space == FEM_COEF_P1 || space == FEM_COEF_P0;
    if (!rule_ok || !space_ok || (dtype != FEM_F32 && dtype != FEM_F64)) return hipErrorInvalidValue;
    auto go = [&](auto dim_c, auto phys_c, auto order_c) -> hipError_t {
        constexpr int D = decltype(dim_c)::value, P = decltype(phys_c)::value, O = decltype(order_c)::value;
        return dtype == FEM_F32 ? launch_jac<D, P, O, float>(rule, space, a, l)
                                : launch_jac<D, P, O, double>(rule, space, a, l);
    };
    auto by_order = [&](auto dim_c, auto phys_c) -> hipError_t {
        if (order == 1) return go(dim_c, phys_c, std::integral_constant<int, 1>());
        if (order == 2) return go(dim_c, phys_c, std::integral_constant<int, 2>());
        return hipErrorInvalidValue;
    };
    auto by_phys = [&](auto dim_c) -> hipError_t {
        switch (phys) {
        case FEM_LAPLACE: return by_order(dim_c, std::integral_constant<int, FEM_LAPLACE>());
        case FEM_ELASTICITY: return by_order(dim_c, std::integral_constant<int, FEM_ELASTICITY>());
        case FEM_MASS: return by_order(dim_c, std::integral_constant<int, FEM_MASS>());
        default: return hipErrorInvalidValue;
        }
    };
    if (dim == 2) return by_phys(std::integral_constant<int, 2>());
    if (dim == 3) return by_phys(std::integral_constant<int, 3>());
    return hipErrorInvalidValue;
}

}  // namespace femq
