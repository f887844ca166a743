// residual_p3.hip -- element residuals of third-order (P3) Lagrange elements,
// their adjoint and element matrices from precomputed affine geometry.
//
// One lane per element, as the P1 and P2 lane kernels: every SoA row
// (inverse Jacobian, det J, the N_b * N_comp closure rows, the coefficient
// rows) is one coalesced access per wave, and the quadrature and basis
// phases run in registers with the basis tabulated at compile time
// (p3_device.hpp). Workgroups hold at most four waves, so the largest
// elements (3D elasticity in FP64) may use the accumulation registers too
// instead of spilling to memory.
//
// Tetrahedra with a gradient term go through their point orbits (P3Tet): 3D
// elasticity takes about 2900 vector instructions and 160 registers in FP32,
// 327 in FP64, where the tabulated products took 4000, 178 and 395; so three
// waves fit a SIMD in FP32. FP32, 600,032 tets, 365 MB: 91 -> 68 us (floor 57);
// FP64, 2^20 tets, 1.28 GB: 283 -> 248 us (floor 198), one wave per SIMD. Their
// adjoint holds the gradient of w once for both outputs and takes u component
// by component (218 registers, and 407 with 38 of them spilled to the
// accumulation registers; 209, and 512 with spills to memory before): 131 ->
// 112 us and 310 -> 237 us at 600,032 tets (floors 109 and 219). Rows at odd words,
// 600,011 tets: residual 152 -> 73 and 219 -> 168 us, adjoint 225 -> 137 and 354 ->
// 259 us, most of it by their stores and workgroup order. 1000 tets, a wave's own
// latency with the call: residual 10.0 -> 8.3 and 11.8 -> 8.8 us.
#include "fem_internal.hpp"
#include "p3_device.hpp"

namespace femq {

// Whether the element is evaluated through its point orbits (P3Tet): the
// tetrahedron's forms with a gradient term. In phases: the gradient of every
// component at all eleven points (99 words for elasticity, where the closure's
// 60 die component by component), the flux in place of the gradient, and the
// sums onto the basis, stored component by component.
template <int DIM, int PHYS>
constexpr bool p3_tet() { return DIM == 3 && Physics<PHYS>::HAS_F1; }

// Gradient of every component at every point from the closure u[b * NC + c].
template <int NC, typename Real>
__device__ __forceinline__ void tet_gradients(const Real* u, const Real* ij, Real (&G)[11][NC][3]) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
        P3Tet::gradients<NC, Real>(u + c, ij, [&](auto q_c, const Real (&g)[3]) {
#pragma unroll
            for (int i = 0; i < 3; ++i) G[decltype(q_c)::value][c][i] = g[i];
        });
}

// Weighted flux at every point in place of the gradient.
template <int PHYS, int NC, typename Real>
__device__ __forceinline__ void tet_flux(Real adj, const Real* aq, Real (&G)[11][NC][3]) {
    constexpr int NCOEF = PHYS == FEM_ELASTICITY ? 2 : 1;
#pragma unroll
    for (int q = 0; q < 11; ++q) {
        Real a[NCOEF];
#pragma unroll
        for (int m = 0; m < NCOEF; ++m) a[m] = (Real(P3Tet::Q::w(q)) * adj) * aq[m * 11 + q];
        p3_weighted_flux<PHYS, NC, Real>(G[q], a);
    }
}

// The sums onto the basis, to the output rows of element e.
template <int NC, bool STREAM_OUT, typename Real>
__device__ __forceinline__ void tet_store(const Real* ij, const Real (&G)[11][NC][3], Real* __restrict__ out, int64_t n,
                                          int64_t e) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        Real r[20];
        P3Tet::scatter<Real>(ij, [&](auto q_c, int i) { return G[decltype(q_c)::value][c][i]; }, r);
#pragma unroll
        for (int b = 0; b < 20; ++b) row_st<STREAM_OUT>(r[b], out + (b * NC + c) * n + e);
    }
}

template <int DIM, int PHYS, typename Real, bool STREAM_OUT>
__global__ void __launch_bounds__(256)
residual_p3_kernel(int64_t n, int place, int space, const Real* __restrict__ inv_j, const Real* __restrict__ det_j,
                   const Real* __restrict__ u, const Real* __restrict__ coef, Real* __restrict__ out) {
    constexpr int RULE = DIM == 2 ? FEM_RULE_TRI6 : FEM_RULE_TET11;
    using E = ElemP3<DIM, PHYS, RULE, FEM_COEF_QUAD>;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = element_block<STREAM_OUT>(place) * blockDim.x + threadIdx.x; e < n; e += stride) {
        Real ij[E::NG], uu[E::NBT], aq[E::NCQ];
        load_rows<E::NG>(inv_j, n, e, ij);
        const Real dj = row_ld(det_j + e);
        load_rows<E::NBT>(u, n, e, uu);
        if constexpr (p3_tet<DIM, PHYS>()) {
            Real G[E::NQ][E::NC][3];
            tet_gradients<E::NC, Real>(uu, ij, G);
            p3_coef_points<DIM, PHYS, RULE, Real>(space, coef, n, e, aq);
            tet_flux<PHYS, E::NC, Real>(fabs(dj), aq, G);
            tet_store<E::NC, STREAM_OUT, Real>(ij, G, out, n, e);
        } else {
            Real r[E::NBT];
            p3_coef_points<DIM, PHYS, RULE, Real>(space, coef, n, e, aq);
            element_residual_p3<DIM, PHYS, RULE, Real>(ij, dj, uu, aq, r);
            store_rows<E::NBT, STREAM_OUT>(out, n, e, r);
        }
    }
}

// du = R(w) (the forms are symmetric) and dcoef, the derivative with respect
// to the coefficient words: the point values mapped back onto the space
// (the transpose of p3_coef_points). Either output may be skipped
// (uniform flags); u is read only for dcoef.
template <int DIM, int PHYS, typename Real, bool STREAM_OUT>
__global__ void __launch_bounds__(256)
backward_p3_kernel(int64_t n, int place, int space, const Real* __restrict__ inv_j, const Real* __restrict__ det_j,
                   const Real* __restrict__ u, const Real* __restrict__ coef, const Real* __restrict__ w,
                   Real* __restrict__ du, Real* __restrict__ dcoef) {
    constexpr int RULE = DIM == 2 ? FEM_RULE_TRI6 : FEM_RULE_TET11;
    using E = ElemP3<DIM, PHYS, RULE, FEM_COEF_QUAD>;
    using Q = RuleP2<DIM, RULE>;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = element_block<STREAM_OUT>(place) * blockDim.x + threadIdx.x; e < n; e += stride) {
        Real ij[E::NG], ww[E::NBT];
        load_rows<E::NG>(inv_j, n, e, ij);
        const Real dj = row_ld(det_j + e);
        load_rows<E::NBT>(w, n, e, ww);
        Real dq[E::NCQ];
        if constexpr (p3_tet<DIM, PHYS>()) {
            Real G[E::NQ][E::NC][3];  // gradients of w
            tet_gradients<E::NC, Real>(ww, ij, G);
            const Real adj = fabs(dj);
            if (dcoef != nullptr) {
                // component c of u against row c of f1(w; e_m): the trace of
                // grad u accumulates, and grad u : (grad w + grad w^T)
#pragma unroll
                for (int f = 0; f < E::NCQ; ++f) dq[f] = Real(0);
#pragma unroll
                for (int c = 0; c < E::NC; ++c) {
                    Real uu[E::NB];
#pragma unroll
                    for (int b = 0; b < E::NB; ++b) uu[b] = row_ld(u + (b * E::NC + c) * n + e);
                    P3Tet::gradients<1, Real>(uu, ij, [&](auto q_c, const Real (&g)[3]) {
                        constexpr int q = decltype(q_c)::value;
                        if constexpr (PHYS == FEM_LAPLACE) {
                            dq[q] = fmadd(g[2], G[q][0][2], fmadd(g[1], G[q][0][1], g[0] * G[q][0][0]));
                        } else {
                            dq[q] += g[c];
#pragma unroll
                            for (int i = 0; i < 3; ++i) dq[E::NQ + q] = fmadd(g[i], G[q][c][i] + G[q][i][c], dq[E::NQ + q]);
                        }
                    });
                }
#pragma unroll
                for (int q = 0; q < E::NQ; ++q) {
                    const Real s = Real(Q::w(q)) * adj;
                    if constexpr (PHYS == FEM_LAPLACE) {
                        dq[q] *= s;
                    } else {
                        dq[q] *= s * ((G[q][0][0] + G[q][1][1]) + G[q][2][2]);
                        dq[E::NQ + q] *= s;
                    }
                }
            }
            if (du != nullptr) {
                Real aq[E::NCQ];
                p3_coef_points<DIM, PHYS, RULE, Real>(space, coef, n, e, aq);
                tet_flux<PHYS, E::NC, Real>(adj, aq, G);
                tet_store<E::NC, STREAM_OUT, Real>(ij, G, du, n, e);
            }
        } else {
            if (du != nullptr) {
                Real aq[E::NCQ], r[E::NBT];
                p3_coef_points<DIM, PHYS, RULE, Real>(space, coef, n, e, aq);
                element_residual_p3<DIM, PHYS, RULE, Real>(ij, dj, ww, aq, r);
                store_rows<E::NBT, STREAM_OUT>(du, n, e, r);
            }
            if (dcoef != nullptr) {
                Real uu[E::NBT];
                load_rows<E::NBT>(u, n, e, uu);
                element_dcoef_points_p3<DIM, PHYS, RULE, Real>(ij, dj, uu, ww, dq);
            }
        }
        if (dcoef != nullptr) {
            if (space == FEM_COEF_QUAD) {
                store_rows<E::NCQ, STREAM_OUT>(dcoef, n, e, dq);
            } else if (space == FEM_COEF_P1) {
#pragma unroll
                for (int m = 0; m < E::NCOEF; ++m)
#pragma unroll
                    for (int v = 0; v < E::NV; ++v) {
                        Real t = Real(0);
#pragma unroll
                        for (int q = 0; q < E::NQ; ++q) t = fmadd(Real(Q::lam(q, v)), dq[m * E::NQ + q], t);
                        row_st<STREAM_OUT>(t, dcoef + (m * E::NV + v) * n + e);
                    }
            } else {
#pragma unroll
                for (int m = 0; m < E::NCOEF; ++m) {
                    Real t = Real(0);
#pragma unroll
                    for (int q = 0; q < E::NQ; ++q) t += dq[m * E::NQ + q];
                    row_st<STREAM_OUT>(t, dcoef + m * n + e);
                }
            }
        }
    }
}

// Element matrices: the three forms are linear in u, so column s of K_e is
// R_e(e_s), the residual of the unit closure e_s = (basis function b_s,
// component c_s). Its value and gradient at a point are phi_{b_s} and
// sum_v dphi_{b_s}/dlam_v g_v in component c_s alone, read from a table
// with the wave-uniform index b_s; the basis phase is the residual's, over
// the rows r <= s only. Column s stores those entries at (r, s) and (s, r),
// so the matrix is exactly symmetric. Columns run in a loop (the arithmetic
// is inlined once); blockIdx.y deals them out where the elements alone leave
// the chip idle (matrix_parts).
__constant__ P3Table<2, FEM_RULE_TRI6> kP3Table2;
__constant__ P3Table<3, FEM_RULE_TET11> kP3Table3;

template <int DIM>
__device__ __forceinline__ const auto& p3_table() {
    if constexpr (DIM == 2) return kP3Table2;
    else return kP3Table3;
}

template <int DIM, int PHYS, typename Real, bool STREAM_OUT>
__global__ void __launch_bounds__(256)
jacobian_p3_kernel(int64_t n, int order, int space, const Real* __restrict__ inv_j, const Real* __restrict__ det_j,
                   const Real* __restrict__ coef, Real* __restrict__ out) {
    constexpr int RULE = DIM == 2 ? FEM_RULE_TRI6 : FEM_RULE_TET11;
    using E = ElemP3<DIM, PHYS, RULE, FEM_COEF_QUAD>;
    using Q = RuleP2<DIM, RULE>;
    using T = P3Basis<DIM, RULE>;
    using P = Physics<PHYS>;
    constexpr int M = E::NBT, NC = E::NC, NV = E::NV, NB = E::NB;
    const auto& tab = p3_table<DIM>();
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = row_block<STREAM_OUT>(order) * blockDim.x + threadIdx.x; e < n; e += stride) {
        Real ij[E::NG], aq[E::NCQ];
        load_rows<E::NG>(inv_j, n, e, ij);
        const Real adj = fabs(row_ld(det_j + e));
        p3_coef_points<DIM, PHYS, RULE, Real>(space, coef, n, e, aq);
        Real g[NV][DIM];
        p2_bary_grads<DIM, Real>(ij, g);
#pragma unroll 1
        for (int s = blockIdx.y; s < M; s += gridDim.y) {
            const int bs = s / NC, cs = s - bs * NC;
            Real r[M];
#pragma unroll
            for (int f = 0; f < M; ++f) r[f] = Real(0);
            unroll_for<0, E::NQ>([&](auto q_c) {
                constexpr int q = decltype(q_c)::value;
                Real uq[NC], gq[NC][DIM];
                if constexpr (P::NEEDS_U) {
                    const Real ph = Real(tab.phi[q][bs]);
#pragma unroll
                    for (int c = 0; c < NC; ++c) uq[c] = c == cs ? ph : Real(0);
                }
                if constexpr (P::HAS_F1) {
                    Real gs[DIM];
#pragma unroll
                    for (int i = 0; i < DIM; ++i) {
                        Real t = Real(tab.dl[q][bs][0]) * g[0][i];
#pragma unroll
                        for (int v = 1; v < NV; ++v) t = fmadd(Real(tab.dl[q][bs][v]), g[v][i], t);
                        gs[i] = t;
                    }
#pragma unroll
                    for (int c = 0; c < NC; ++c)
#pragma unroll
                        for (int i = 0; i < DIM; ++i) gq[c][i] = c == cs ? gs[i] : Real(0);
                }
                Real a[E::NCOEF];
#pragma unroll
                for (int m = 0; m < E::NCOEF; ++m) a[m] = aq[m * E::NQ + q];
                Real f0[NC], f1[NC][DIM];
                P::template point<DIM, Real>(uq, gq, a, f0, f1);
                const Real w = Real(Q::w(q)) * adj;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    if constexpr (P::HAS_F1) {
                        Real h[NV];
#pragma unroll
                        for (int v = 0; v < NV; ++v) {
                            Real t = g[v][0] * f1[c][0];
#pragma unroll
                            for (int i = 1; i < DIM; ++i) t = fmadd(g[v][i], f1[c][i], t);
                            h[v] = w * t;
                        }
                        unroll_for<0, NB>([&](auto b_c) {
                            constexpr int b = decltype(b_c)::value;
                            if (b * NC + c <= s) {
                                unroll_for<0, NV>([&](auto v_c) {
                                    constexpr int v = decltype(v_c)::value;
                                    constexpr double d = T::dl(q, b, v);
                                    if constexpr (d != 0.0) r[b * NC + c] = fmadd(Real(d), h[v], r[b * NC + c]);
                                });
                            }
                        });
                    }
                    if constexpr (P::HAS_F0) {
                        const Real sf = w * f0[c];
                        unroll_for<0, NB>([&](auto b_c) {
                            constexpr int b = decltype(b_c)::value;
                            if (b * NC + c <= s) r[b * NC + c] = fmadd(Real(T::phi(q, b)), sf, r[b * NC + c]);
                        });
                    }
                }
            });
#pragma unroll
            for (int f = 0; f < M; ++f) {
                if (f <= s) {
                    row_st<STREAM_OUT>(r[f], out + (int64_t)(f * M + s) * n + e);
                    row_st<STREAM_OUT>(r[f], out + (int64_t)(s * M + f) * n + e);
                }
            }
        }
    }
}

template <int DIM, int PHYS, typename Real>
static hipError_t launch_jac(int space, const JacobianArgs& a, const Launch& l) {
    constexpr int M = ElemP3<DIM, PHYS, DIM == 2 ? FEM_RULE_TRI6 : FEM_RULE_TET11, FEM_COEF_QUAD>::NBT;
    const auto k = l.stream_out ? jacobian_p3_kernel<DIM, PHYS, Real, true> : jacobian_p3_kernel<DIM, PHYS, Real, false>;
    // Two waves per SIMD, which is what the registers hold; the FP32 Laplacian is
    // bound by its arithmetic and holds four (100,003 tets: 67 us with 2048 waves
    // wanted, 53 with 4096). No more than that many, so that all shares run at once (3D
    // elasticity FP32, 10,240 tets: 40 us with 12, 57 with 13), but whole lines of up to
    // two thirds as many waves take two shares (2D elasticity FP32, 81,920 triangles 37
    // and 30 us, 3D mass FP32 33 and 30; at odd words that loses: 3D Laplacian FP32,
    // 163,859 tets 77 and 83).
    int64_t want = PHYS == FEM_LAPLACE && std::is_same<Real, float>::value ? 4096 : 2048;
    const int64_t waves = blocks_for_lanes(l, a.n) * (l.block / 64);
    if (l.stream_out && 2 * waves > want && 3 * waves <= 2 * want) want = 2 * waves;
    hipLaunchKernelGGL(k, dim3(l.grid, matrix_parts(l, a.n, M, want)), dim3(l.block), 0, l.stream, a.n, l.order, space,
                       static_cast<const Real*>(a.inv_j), static_cast<const Real*>(a.det_j),
                       static_cast<const Real*>(a.coef), static_cast<Real*>(a.out));
    return hipGetLastError();
}

template <int DIM, int PHYS, typename Real>
static hipError_t launch_bwd(int space, const BackwardArgs& a, const Launch& l) {
    const auto k = l.stream_out ? backward_p3_kernel<DIM, PHYS, Real, true> : backward_p3_kernel<DIM, PHYS, Real, false>;
    hipLaunchKernelGGL(k, dim3(l.grid), dim3(l.block), 0, l.stream, a.n, l.place(), space,
                       static_cast<const Real*>(a.inv_j), static_cast<const Real*>(a.det_j),
                       static_cast<const Real*>(a.u), static_cast<const Real*>(a.coef), static_cast<const Real*>(a.w),
                       static_cast<Real*>(a.du), static_cast<Real*>(a.dcoef));
    return hipGetLastError();
}

template <int DIM, int PHYS, typename Real>
static hipError_t launch_fwd(int space, const ResidualArgs& a, const Launch& l) {
    const auto k = l.stream_out ? residual_p3_kernel<DIM, PHYS, Real, true> : residual_p3_kernel<DIM, PHYS, Real, false>;
    hipLaunchKernelGGL(k, dim3(l.grid), dim3(l.block), 0, l.stream, a.n, l.place(), space,
                       static_cast<const Real*>(a.inv_j), static_cast<const Real*>(a.det_j),
                       static_cast<const Real*>(a.u), static_cast<const Real*>(a.coef), static_cast<Real*>(a.out));
    return hipGetLastError();
}

// Runtime (dim, physics, dtype) to a kernel instance; the rule is the
// degree-4 rule of the dimension (checked by the caller), the space a
// kernel argument.
template <typename F>
static hipError_t p3_dispatch(int dim, int phys, int space, int dtype, const F& f) {
    if (space != FEM_COEF_QUAD && space != FEM_COEF_P1 && space != FEM_COEF_P0) return hipErrorInvalidValue;
    auto by_phys = [&](auto dim_c) -> hipError_t {
        constexpr int D = decltype(dim_c)::value;
        auto go = [&](auto phys_c) -> hipError_t {
            constexpr int P = decltype(phys_c)::value;
            return dtype == FEM_F32 ? f.template operator()<D, P, float>() : f.template operator()<D, P, double>();
        };
        switch (phys) {
        case FEM_LAPLACE: return go(std::integral_constant<int, FEM_LAPLACE>());
        case FEM_ELASTICITY: return go(std::integral_constant<int, FEM_ELASTICITY>());
        case FEM_MASS: return go(std::integral_constant<int, FEM_MASS>());
        default: return hipErrorInvalidValue;
        }
    };
    if (dim == 2) return by_phys(std::integral_constant<int, 2>());
    if (dim == 3) return by_phys(std::integral_constant<int, 3>());
    return hipErrorInvalidValue;
}

struct P3Fwd {
    int space;
    const ResidualArgs& a;
    const Launch& l;
    template <int D, int P, typename Real>
    hipError_t operator()() const { return launch_fwd<D, P, Real>(space, a, l); }
};

struct P3Bwd {
    int space;
    const BackwardArgs& a;
    const Launch& l;
    template <int D, int P, typename Real>
    hipError_t operator()() const { return launch_bwd<D, P, Real>(space, a, l); }
};

struct P3Jac {
    int space;
    const JacobianArgs& a;
    const Launch& l;
    template <int D, int P, typename Real>
    hipError_t operator()() const { return launch_jac<D, P, Real>(space, a, l); }
};

hipError_t launch_jacobian_p3(int dim, int phys, int space, int dtype, const JacobianArgs& a, const Launch& l) {
    return p3_dispatch(dim, phys, space, dtype, P3Jac{space, a, l});
}

hipError_t launch_residual_p3(int dim, int phys, int space, int dtype, const ResidualArgs& a, const Launch& l) {
    return p3_dispatch(dim, phys, space, dtype, P3Fwd{space, a, l});
}

hipError_t launch_backward_p3(int dim, int phys, int space, int dtype, const BackwardArgs& a, const Launch& l) {
    return p3_dispatch(dim, phys, space, dtype, P3Bwd{space, a, l});
}

}  // namespace femq
