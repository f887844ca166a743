// backward_lane.hip -- adjoint of the element residual, one lane per element.
//
// For L = sum_e w_e . R_e: du_e = R_e(u := w_e) because every supported form
// is a symmetric bilinear form in (u, test function), and dcoef at each
// quadrature point is the weighted pointwise derivative of f0/f1 with respect
// to the coefficient (the forms are linear in the coefficients). Same
// coalesced V-wide SoA access as the forward kernel; du and dcoef are
// optional (wave-uniform branches), and u is only read when dcoef is wanted.
#include "fem_device.hpp"
#include "fem_internal.hpp"

namespace femq {

template <int DIM, int PHYS, int RULE, typename Real, int V, bool STREAM_OUT>
__global__ void __launch_bounds__(512)
backward_lane_kernel(int64_t n, int place, const Real* __restrict__ inv_j, const Real* __restrict__ det_j,
                     const Real* __restrict__ u, const Real* __restrict__ coef,
                     const Real* __restrict__ w, Real* __restrict__ du, Real* __restrict__ dcoef) {
    using E = Elem<DIM, PHYS, RULE>;
    const int64_t nchunk = (n + V - 1) / V;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const bool want_du = du != nullptr;
    const bool want_dc = dcoef != nullptr;
    for (int64_t ch = element_block<STREAM_OUT>(place) * blockDim.x + threadIdx.x; ch < nchunk; ch += stride) {
        for_chunk<V>(ch * V, n, [&](auto width, int64_t e) {
            constexpr int W = decltype(width)::value;
            Real rij[E::NG][W], rdj[1][W], rw[E::NBT][W];
            load_rows_v<E::NG>(inv_j, n, e, rij);
            load_rows_v<1>(det_j, n, e, rdj);
            load_rows_v<E::NBT>(w, n, e, rw);
            if (want_du) {
                Real rcf[E::NCQ][W], rr[E::NBT][W];
                load_rows_v<E::NCQ>(coef, n, e, rcf);
                lane_residual<DIM, PHYS, RULE, Real>(rij, rdj, rw, rcf, rr);
                store_rows_v<E::NBT, STREAM_OUT>(du, n, e, rr);
            }
            if (want_dc) {
                Real ru[E::NBT][W], rd[E::NCQ][W];
                load_rows_v<E::NBT>(u, n, e, ru);
#pragma unroll
                for (int v = 0; v < W; ++v) {
                    Real ij[E::NG], uu[E::NBT], ww[E::NBT], d[E::NCQ];
#pragma unroll
                    for (int f = 0; f < E::NG; ++f) ij[f] = rij[f][v];
#pragma unroll
                    for (int f = 0; f < E::NBT; ++f) {
                        uu[f] = ru[f][v];
                        ww[f] = rw[f][v];
                    }
                    element_dcoef<DIM, PHYS, RULE, Real>(ij, rdj[0][v], uu, ww, d);
#pragma unroll
                    for (int f = 0; f < E::NCQ; ++f) rd[f][v] = d[f];
                }
                store_rows_v<E::NCQ, STREAM_OUT>(dcoef, n, e, rd);
            }
        });
    }
}

template <int DIM, int PHYS, int RULE, typename Real>
static hipError_t launch_v(const BackwardArgs& a, const Launch& l) {
    const Real* ij = static_cast<const Real*>(a.inv_j);
    const Real* dj = static_cast<const Real*>(a.det_j);
    const Real* u = static_cast<const Real*>(a.u);
    const Real* cf = static_cast<const Real*>(a.coef);
    const Real* w = static_cast<const Real*>(a.w);
    Real* du = static_cast<Real*>(a.du);
    Real* dc = static_cast<Real*>(a.dcoef);
    auto go = [&](auto vec_c) {
        constexpr int V = decltype(vec_c)::value;
        const auto k = l.stream_out ? backward_lane_kernel<DIM, PHYS, RULE, Real, V, true>
                               : backward_lane_kernel<DIM, PHYS, RULE, Real, V, false>;
        hipLaunchKernelGGL(k, dim3(l.grid), dim3(l.block), 0, l.stream, a.n, l.place(), ij, dj, u, cf, w, du, dc);
    };
    switch (l.vec) {
    case 1: go(std::integral_constant<int, 1>()); break;
    case 2: go(std::integral_constant<int, 2>()); break;
    case 4: go(std::integral_constant<int, 4>()); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int DIM, int PHYS, int RULE>
static hipError_t launch_t(int dtype, const BackwardArgs& a, const Launch& l) {
    return dtype == FEM_F32 ? launch_v<DIM, PHYS, RULE, float>(a, l) : launch_v<DIM, PHYS, RULE, double>(a, l);
}

struct BackwardDispatch {
    int dtype;
    const BackwardArgs& a;
    const Launch& l;
    template <int D, int P, int S>
    hipError_t operator()() const { return launch_t<D, P, S>(dtype, a, l); }
};

hipError_t launch_backward_lane(int dim, int phys, int rule, int space, int dtype, const BackwardArgs& a,
                               const Launch& l) {
    const BackwardDispatch f{dtype, a, l};
    return dispatch_element(dim, phys, rule, space, f, hipErrorInvalidValue);
}

}  // namespace femq
