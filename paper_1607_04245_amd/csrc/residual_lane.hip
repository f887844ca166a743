// residual_lane.hip -- element residual kernels, one lane per element.
//
// Each lane owns V consecutive elements. Every structure-of-arrays row is
// read with one V-wide vector load per lane, so a wavefront reads 64*V
// consecutive words of a row at once (fully coalesced). Rows may start on any
// word: the rows of an odd element count do, and V = 4 is there for them in FP32,
// since a wave then shares only the two lines at the ends of its 1 KB with other
// waves (P1 3D Laplacian FP32, 2,272,267 tets: 50.4 us with one element per lane and
// streaming stores, 36.8 with plain stores in runs of workgroups, 35.0 with four
// elements per lane, floor 31.0). The quadrature phase (pointwise f0/f1 at every
// point) and the basis phase (sum back onto the basis functions) run in
// registers, so no value crosses lanes and no reduction is needed; the paper's
// concern about per-thread storage (Section 1) does not bind on gfx950, whose
// lanes hold up to 512 VGPRs. Grid-stride over chunks of V elements.
#include "fem_device.hpp"
#include "fem_internal.hpp"

namespace femq {

template <int DIM, int PHYS, int RULE, typename Real, int V, bool STREAM_OUT>
__global__ void __launch_bounds__(512)
residual_lane_kernel(int64_t n, int place, const Real* __restrict__ inv_j, const Real* __restrict__ det_j,
                     const Real* __restrict__ u, const Real* __restrict__ coef,
                     Real* __restrict__ out) {
    using E = Elem<DIM, PHYS, RULE>;
    const int64_t nchunk = (n + V - 1) / V;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t ch = element_block<STREAM_OUT>(place) * blockDim.x + threadIdx.x; ch < nchunk; ch += stride) {
        for_chunk<V>(ch * V, n, [&](auto width, int64_t e) {
            constexpr int W = decltype(width)::value;
            Real rij[E::NG][W], rdj[1][W], ru[E::NBT][W], rcf[E::NCQ][W], rr[E::NBT][W];
            load_rows_v<E::NG>(inv_j, n, e, rij);
            load_rows_v<1>(det_j, n, e, rdj);
            load_rows_v<E::NBT>(u, n, e, ru);
            load_rows_v<E::NCQ>(coef, n, e, rcf);
            lane_residual<DIM, PHYS, RULE, Real>(rij, rdj, ru, rcf, rr);
            store_rows_v<E::NBT, STREAM_OUT>(out, n, e, rr);
        });
    }
}

template <int DIM, int PHYS, int RULE, typename Real>
static hipError_t launch_v(const ResidualArgs& a, const Launch& l) {
    const Real* ij = static_cast<const Real*>(a.inv_j);
    const Real* dj = static_cast<const Real*>(a.det_j);
    const Real* u = static_cast<const Real*>(a.u);
    const Real* cf = static_cast<const Real*>(a.coef);
    Real* out = static_cast<Real*>(a.out);
    auto go = [&](auto vec_c) {
        constexpr int V = decltype(vec_c)::value;
        const auto k = l.stream_out ? residual_lane_kernel<DIM, PHYS, RULE, Real, V, true>
                               : residual_lane_kernel<DIM, PHYS, RULE, Real, V, false>;
        hipLaunchKernelGGL(k, dim3(l.grid), dim3(l.block), 0, l.stream, a.n, l.place(), ij, dj, u, cf, out);
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
static hipError_t launch_t(int dtype, const ResidualArgs& a, const Launch& l) {
    return dtype == FEM_F32 ? launch_v<DIM, PHYS, RULE, float>(a, l) : launch_v<DIM, PHYS, RULE, double>(a, l);
}

struct LaneDispatch {
    int dtype;
    const ResidualArgs& a;
    const Launch& l;
    template <int D, int P, int S>
    hipError_t operator()() const { return launch_t<D, P, S>(dtype, a, l); }
};

hipError_t launch_residual_lane(int dim, int phys, int rule, int space, int dtype, const ResidualArgs& a,
                               const Launch& l) {
    const LaneDispatch f{dtype, a, l};
    return dispatch_element(dim, phys, rule, space, f, hipErrorInvalidValue);
}

}  // namespace femq
