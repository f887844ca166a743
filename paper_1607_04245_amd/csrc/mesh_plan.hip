// mesh_plan.hip -- a per-mesh plan of the distinct vertices of every
// 64-element tile, and the from-mesh residual kernels that use it.
//
// The fused from-mesh kernels (mesh_kernel.hpp) let every lane gather the
// vertices of its own element: d+1 vertex records per element, while the
// elements of a 64-element tile of a conforming mesh share most of their
// vertices (47 distinct vertices for 256 references on a tetrahedral grid).
// The per-lane gathers, not the bytes, bound those kernels. A plan, built
// once per mesh from the connectivity, lists each tile's distinct vertices
// (ascending) and, per element, the position of each of its vertices in
// that list (one byte each, packed in 32 bits, in place of the 4(d+1)-byte
// connectivity row). The planned kernel gives each wave one tile: the lanes
// load the tile's distinct vertex records once (coordinates; in the gather
// form also u and a P1 coefficient) into LDS, then every lane reads its
// element's vertices from LDS and runs the fused kernel's element arithmetic
// on them, so the element vectors are bitwise those of
// fem_integrate_residual_mesh / fem_integrate_residual_gather.
//
// The plan is built on the device, one wave per tile: the wave sorts its
// tile's vertex indices in registers, ballots number the distinct ones, and
// each element finds its vertices in that list. A first pass counts, a scan
// places the lists, a second pass writes them (sorting again, 12 us for
// 400,003 tets, costs less than scratch for the lists of the first pass). The
// build takes 65 us there, two thirds of it allocations and the wait for the
// sizes, where a host sort of every tile took 13 ms. It validates every vertex
// index, so the planned kernels need no index checks.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <new>

#include "mesh_kernel.hpp"

struct fem_mesh_plan {
    int dim = 0;
    int device = 0;
    int max_tile = 0;                // distinct vertices of the fullest tile (<= 64 (dim+1))
    int64_t n_elem = 0;
    int64_t n_vert = 0;
    int64_t n_tiles = 0;
    int64_t total = 0;               // entries of tile_verts
    void* block = nullptr;           // the allocation that holds tile_off and lidx
    int64_t* tile_off = nullptr;     // [n_tiles + 1]: tile t's vertices are tile_verts[tile_off[t] ..)
    int32_t* tile_verts = nullptr;   // [tile_off[n_tiles]], ascending within a tile
    uint32_t* lidx = nullptr;        // [n_elem]: byte b = position of the element's vertex b in its tile's list
};

namespace femq {

constexpr int kPlanTile = 64;

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wave (the whole workgroup) per TPW consecutive tiles, whose loads are
// all issued before the first element is finished (two in the gather form on
// triangles, one otherwise). LDS
// holds, per tile, maxc x DIM coordinates (FP64), then, after all tiles'
// coordinates, maxc x (NU + NK) values of u and of a P1 coefficient (gather
// form).
template <int DIM, int PHYS, int RULE, typename Real, bool GATHER, bool STORE_GEOM, int TPW, bool STREAM_OUT>
__global__ void __launch_bounds__(64)
residual_planned_kernel(int64_t n, int64_t n_tiles, const int64_t* __restrict__ tile_off,
                        const int32_t* __restrict__ tile_verts, const uint32_t* __restrict__ lidx,
                        const double* __restrict__ X, const Real* __restrict__ u, const Real* __restrict__ coef,
                        Real* __restrict__ out, Real* __restrict__ inv_j, Real* __restrict__ det_j,
                        int32_t* __restrict__ counts, int maxc, int order) {
    using E = Elem<DIM, PHYS, RULE>;
    constexpr bool CV = coef_per_vertex<DIM, PHYS, RULE, GATHER>();
    constexpr int NU = GATHER ? E::NC : 0, NK = CV ? E::NCOEF : 0, NR = NU + NK;
    extern __shared__ double plan_lds[];
    double* xs = plan_lds;
    Real* vs = reinterpret_cast<Real*>(plan_lds + (int64_t)TPW * maxc * DIM);
    const int lane = threadIdx.x;
    int ndeg = 0, npoor = 0;
    for (int64_t t0 = row_block<STREAM_OUT>(order) * TPW; t0 < n_tiles; t0 += (int64_t)gridDim.x * TPW) {
        int64_t off[TPW], e[TPW];
        int cnt[TPW];
        uint32_t li[TPW];
        Real uu[TPW][E::NBT], cf[TPW][E::NCQ];
#pragma unroll
        for (int k = 0; k < TPW; ++k) {
            // a tile past the end is skipped: no records, masked stores
            const bool live = t0 + k < n_tiles;
            const int64_t t = live ? t0 + k : n_tiles - 1;
            off[k] = tile_off[t];
            cnt[k] = live ? (int)(tile_off[t + 1] - off[k]) : 0;
            // per-element streams, independent of the vertex records
            e[k] = (t0 + k) * kPlanTile + lane;
            const int64_t ec = e[k] < n ? e[k] : n - 1;
            li[k] = __builtin_nontemporal_load(lidx + ec);
            if constexpr (!GATHER) {
#pragma unroll
                for (int f = 0; f < E::NBT; ++f) uu[k][f] = __builtin_nontemporal_load(u + f * n + ec);
            }
            if constexpr (!CV) {
#pragma unroll
                for (int f = 0; f < E::NCQ; ++f) cf[k][f] = __builtin_nontemporal_load(coef + f * n + ec);
            }
        }
        // the tiles' distinct vertex records, once each (a version that
        // issued all of a lane's record loads before its first LDS store
        // measured slower on tetrahedra and barely faster on triangles)
#pragma unroll
        for (int k = 0; k < TPW; ++k) {
            double* xk = xs + (int64_t)k * maxc * DIM;
            Real* vk = vs + (int64_t)k * maxc * NR;
            for (int j = lane; j < cnt[k]; j += kPlanTile) {
                const int64_t v = tile_verts[off[k] + j];
#pragma unroll
                for (int i = 0; i < DIM; ++i) xk[j * DIM + i] = X[v * DIM + i];
                if constexpr (GATHER) {
#pragma unroll
                    for (int c = 0; c < E::NC; ++c) vk[j * NR + c] = u[v * E::NC + c];
                }
                if constexpr (CV) {
#pragma unroll
                    for (int m = 0; m < E::NCOEF; ++m) vk[j * NR + NU + m] = coef[v * E::NCOEF + m];
                }
            }
        }
        wave_sync();
#pragma unroll
        for (int k = 0; k < TPW; ++k) {
            const double* xk = xs + (int64_t)k * maxc * DIM;
            const Real* vk = vs + (int64_t)k * maxc * NR;
            double x[DIM + 1][DIM];
#pragma unroll
            for (int b = 0; b <= DIM; ++b) {
                const int l = (int)((li[k] >> (8 * b)) & 255u);
#pragma unroll
                for (int i = 0; i < DIM; ++i) x[b][i] = xk[l * DIM + i];
                if constexpr (GATHER) {
#pragma unroll
                    for (int c = 0; c < E::NC; ++c) uu[k][b * E::NC + c] = vk[l * NR + c];
                }
                if constexpr (CV) {
#pragma unroll
                    for (int m = 0; m < E::NCOEF; ++m) cf[k][m * E::NB + b] = vk[l * NR + NU + m];
                }
            }
            mesh_element_finish<DIM, PHYS, RULE, Real, STORE_GEOM, STREAM_OUT>(e[k] < n, e[k], n, true, x, uu[k], cf[k], out,
                                                                   inv_j, det_j, ndeg, npoor);
        }
        wave_sync();  // every lane has read the tiles before the next ones are staged
    }
    add_counts(counts, ndeg, npoor);
}

// The geometry alone through the plan: coordinates staged as above, then
// the epilogue of fem_geometry, so the outputs are bitwise its outputs.
template <int DIM, typename Out, bool STREAM_OUT>
__global__ void __launch_bounds__(64)
geometry_planned_kernel(int64_t n, int64_t n_tiles, const int64_t* __restrict__ tile_off,
                        const int32_t* __restrict__ tile_verts, const uint32_t* __restrict__ lidx,
                        const double* __restrict__ X, Out* __restrict__ inv_j, Out* __restrict__ det_j,
                        int32_t* __restrict__ counts, int order) {
    extern __shared__ double plan_lds[];
    const int lane = threadIdx.x;
    int ndeg = 0, npoor = 0;
    for (int64_t t = row_block<STREAM_OUT>(order); t < n_tiles; t += gridDim.x) {
        const int64_t off = tile_off[t];
        const int cnt = (int)(tile_off[t + 1] - off);
        const int64_t e = t * kPlanTile + lane, ec = e < n ? e : n - 1;
        const uint32_t li = __builtin_nontemporal_load(lidx + ec);
        for (int j = lane; j < cnt; j += kPlanTile) {
            const int64_t v = tile_verts[off + j];
#pragma unroll
            for (int i = 0; i < DIM; ++i) plan_lds[j * DIM + i] = X[v * DIM + i];
        }
        wave_sync();
        double x[DIM + 1][DIM];
#pragma unroll
        for (int b = 0; b <= DIM; ++b) {
            const int l = (int)((li >> (8 * b)) & 255u);
#pragma unroll
            for (int i = 0; i < DIM; ++i) x[b][i] = plan_lds[l * DIM + i];
        }
        geometry_finish<DIM, STREAM_OUT, Out>(e < n, e, n, true, x, inv_j, det_j, ndeg, npoor);
        wave_sync();
    }
    add_counts(counts, ndeg, npoor);
}

// ------------------------------------------------------------- plan build --

constexpr uint32_t kNoVertex = 0xFFFFFFFFu;   // sorts past every vertex index

// Ascending bitonic sort of the wave's 256 keys, key 4 * lane + r in k[r].
__device__ __forceinline__ void wave_sort256(uint32_t (&k)[4], int lane) {
#pragma unroll
    for (int size = 2; size <= 256; size <<= 1) {
#pragma unroll
        for (int j = size >> 1; j > 0; j >>= 1) {
            if (j >= 4) {
                const bool low = (lane & (j >> 2)) == 0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool up = ((4 * lane + r) & size) == 0;
                    const uint32_t o = __shfl_xor(k[r], j >> 2, 64);
                    k[r] = up == low ? min(k[r], o) : max(k[r], o);
                }
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (r & j) continue;
                    const bool up = ((4 * lane + r) & size) == 0;
                    const uint32_t a = k[r], b = k[r | j];
                    k[r] = up ? min(a, b) : max(a, b);
                    k[r | j] = up ? max(a, b) : min(a, b);
                }
            }
        }
    }
}

// One wave per tile (four tiles per workgroup). WRITE false: word[t] = number
// of distinct vertices, plus 2^16 times the number of indices outside
// [0, n_vert). WRITE true: the tile's list at tile_verts[word[t] ..) and every
// element's positions in it.
template <int NB, bool WRITE>
__global__ void __launch_bounds__(256)
mesh_plan_kernel(int64_t n, int64_t n_vert, int64_t n_tiles, const int32_t* __restrict__ conn, int64_t* __restrict__ word,
                 int32_t* __restrict__ tile_verts, uint32_t* __restrict__ lidx) {
    __shared__ uint32_t lists[4][kPlanTile * 4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t* list = lists[wave];
    for (int64_t t = (int64_t)blockIdx.x * 4 + wave; t < n_tiles; t += (int64_t)gridDim.x * 4) {
        const int64_t e = t * kPlanTile + lane;
        uint32_t v[NB], k[4] = {kNoVertex, kNoVertex, kNoVertex, kNoVertex};
        int bad = 0;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int32_t x = e < n ? conn[e * NB + b] : 0;
            bad += (int)((e < n) & ((x < 0) | ((int64_t)x >= n_vert)));
            v[b] = k[b] = e < n ? (uint32_t)x : kNoVertex;
        }
        wave_sort256(k, lane);
        const uint32_t before = __shfl_up(k[3], 1, 64);
        bool first[4];
        int rank = 0, cnt = 0;   // distinct keys below 4 * lane, and of the tile
        const uint64_t below = ((uint64_t)1 << lane) - 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool other = r > 0 ? k[r] != k[r > 0 ? r - 1 : 0] : (lane == 0) | (k[0] != before);
            first[r] = other & (k[r] != kNoVertex);
            const uint64_t m = __ballot(first[r]);
            rank += __popcll(m & below);
            cnt += __popcll(m);
        }
        if constexpr (!WRITE) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) bad += __shfl_xor(bad, off, 64);
            if (lane == 0) word[t] = (int64_t)cnt | (int64_t)bad << 16;
        } else {
            const int64_t base = word[t];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (first[r]) {
                    list[rank] = k[r];
                    tile_verts[base + rank] = (int32_t)k[r];
                    ++rank;
                }
            }
            wave_sync();
            uint32_t packed = 0;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                int lo = 0, len = cnt;   // lower bound of v[b], which is in the list
                while (len > 0) {
                    const int half = len >> 1;
                    const bool right = list[lo + half] < v[b];
                    lo = right ? lo + half + 1 : lo;
                    len = right ? len - half - 1 : half;
                }
                packed |= (uint32_t)lo << (8 * b);
            }
            if (e < n) lidx[e] = packed;
            wave_sync();   // the list is read before the next tile's is written
        }
    }
}

struct MeshPlanTotals {
    int64_t total, bad;
    int max_tile;
};

// Turns the counts of the first pass into list offsets in place (word[n_tiles]
// = the total) and sums them up. One workgroup walks the tiles: 64 elements
// each, so its 4096 counts per step are 2^18 elements.
__global__ void __launch_bounds__(1024)
mesh_plan_scan_kernel(int64_t n_tiles, int64_t* __restrict__ word, MeshPlanTotals* __restrict__ out) {
    __shared__ int64_t wave_sum[16], wave_bad[16];
    __shared__ int wave_max[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t run = 0, bad = 0;
    int most = 0;
    for (int64_t t0 = 0; t0 < n_tiles; t0 += 4096) {
        const int64_t t = t0 + 4 * (int64_t)threadIdx.x;
        int c[4];
        int64_t own = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t w = t + r < n_tiles ? word[t + r] : 0;
            c[r] = (int)(w & 0xFFFF);
            bad += w >> 16;
            most = max(most, c[r]);
            own += c[r];
        }
        int64_t scan = own;   // inclusive over the wave
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int64_t o = __shfl_up(scan, off, 64);
            if (lane >= off) scan += o;
        }
        if (lane == 63) wave_sum[wave] = scan;
        __syncthreads();
        int64_t at = run + scan - own;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            if (w < wave) at += wave_sum[w];
            run += wave_sum[w];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (t + r < n_tiles) word[t + r] = at;
            at += c[r];
        }
        __syncthreads();   // wave_sum is read before the next step writes it
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        bad += __shfl_xor(bad, off, 64);
        most = max(most, __shfl_xor(most, off, 64));
    }
    if (lane == 0) { wave_bad[wave] = bad; wave_max[wave] = most; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) { bad += wave_bad[w]; most = max(most, wave_max[w]); }
        word[n_tiles] = run;
        *out = MeshPlanTotals{run, bad, most};
    }
}

template <int NB, bool WRITE>
static hipError_t launch_mesh_plan(const fem_mesh_plan* p, const int32_t* conn, hipStream_t s) {
    const int64_t grid = std::min<int64_t>((p->n_tiles + 3) / 4, (int64_t)1 << 22);
    hipLaunchKernelGGL((mesh_plan_kernel<NB, WRITE>), dim3((unsigned)grid), dim3(256), 0, s, p->n_elem, p->n_vert,
                       p->n_tiles, conn, p->tile_off, p->tile_verts, p->lidx);
    return hipGetLastError();
}

struct PlannedArgs {
    const fem_mesh_plan* p;
    const double* coords;
    const void* u;
    const void* coef;
    void* out;
    void* inv_j;
    void* det_j;
    int32_t* counts;
    int dtype;
    hipStream_t stream;
};

template <int DIM, int PHYS, int RULE, typename Real, bool GATHER>
static hipError_t launch_planned_t(const PlannedArgs& a) {
    using E = Elem<DIM, PHYS, RULE>;
    constexpr bool CV = coef_per_vertex<DIM, PHYS, RULE, GATHER>();
    constexpr int NR = (GATHER ? E::NC : 0) + (CV ? E::NCOEF : 0);
    // measured: two tiles per wave pay in the triangle gather form only
    constexpr int TPW = (DIM == 2 && GATHER) ? 2 : 1;
    const int maxc = std::max(a.p->max_tile, 1);
    const size_t lds = (size_t)TPW * maxc * (DIM * sizeof(double) + NR * sizeof(Real));
    const int64_t grid =
        std::min<int64_t>(std::max<int64_t>((a.p->n_tiles + TPW - 1) / TPW, 1), (int64_t)1 << 30);
    const bool whole = whole_lines(a.p->n_elem, sizeof(Real), {a.out, a.inv_j, a.det_j});
    auto go = [&](auto geom_c, auto whole_c) {
        hipLaunchKernelGGL((residual_planned_kernel<DIM, PHYS, RULE, Real, GATHER, decltype(geom_c)::value, TPW,
                                                    decltype(whole_c)::value>),
                           dim3((unsigned)grid), dim3(64), lds, a.stream, a.p->n_elem, a.p->n_tiles, a.p->tile_off,
                           a.p->tile_verts, a.p->lidx, a.coords, static_cast<const Real*>(a.u),
                           static_cast<const Real*>(a.coef), static_cast<Real*>(a.out), static_cast<Real*>(a.inv_j),
                           static_cast<Real*>(a.det_j), a.counts, maxc, whole ? kOrderLaunch : kOrderXcd);
    };
    const std::true_type yes;
    const std::false_type no;
    if (a.inv_j != nullptr) whole ? go(yes, yes) : go(yes, no);
    else whole ? go(no, yes) : go(no, no);
    return hipGetLastError();
}

template <bool GATHER>
struct PlannedDispatch {
    const PlannedArgs& a;
    template <int D, int P, int S>
    hipError_t operator()() const {
        return a.dtype == FEM_F32 ? launch_planned_t<D, P, S, float, GATHER>(a)
                                  : launch_planned_t<D, P, S, double, GATHER>(a);
    }
};

static void mesh_plan_free(fem_mesh_plan* p) {
    if (!p) return;
    if (p->block) (void)hipFree(p->block);
    if (p->tile_verts) (void)hipFree(p->tile_verts);
    delete p;
}

static fem_status planned_common(const char* fn, const fem_mesh_plan* plan, int physics, int rule, int coef_space,
                                 int dtype, const double* coords, const void* u, const void* coef, void* out,
                                 const void* inv_j, const void* det_j) {
    if (!plan) { set_error("%s: NULL plan", fn); return FEM_ERR_INVALID_ARG; }
    const int dim = plan->dim;
    if (physics != FEM_LAPLACE && physics != FEM_ELASTICITY && physics != FEM_MASS) {
        set_error("%s: unknown physics %d", fn, physics);
        return FEM_ERR_UNSUPPORTED;
    }
    const bool rule_ok = rule == FEM_RULE_CENTROID || (dim == 2 ? rule == FEM_RULE_TRI3 : rule == FEM_RULE_TET4);
    if (!rule_ok) { set_error("%s: rule %d is not defined in %dD", fn, rule, dim); return FEM_ERR_UNSUPPORTED; }
    if (coef_space != FEM_COEF_QUAD && coef_space != FEM_COEF_P1 && coef_space != FEM_COEF_P0) {
        set_error("%s: unknown coefficient space %d", fn, coef_space);
        return FEM_ERR_UNSUPPORTED;
    }
    if (dtype != FEM_F32 && dtype != FEM_F64) { set_error("%s: unknown dtype %d", fn, dtype); return FEM_ERR_UNSUPPORTED; }
    if (plan->n_elem == 0) return FEM_OK;
    if (!coords || !u || !coef || !out || (!inv_j) != (!det_j)) {
        set_error("%s: NULL array (inv_j and det_j must both be set or both NULL)", fn);
        return FEM_ERR_INVALID_ARG;
    }
    int dev = 0;
    if (hipGetDevice(&dev) == hipSuccess && dev != plan->device) {
        set_error("%s: the plan was built on device %d, current device is %d", fn, plan->device, dev);
        return FEM_ERR_INVALID_ARG;
    }
    return FEM_OK;
}

}  // namespace femq

using namespace femq;

extern "C" {

fem_status fem_mesh_plan_create(int dim, int64_t n_elem, int64_t n_vert, const int32_t* conn, void* stream,
                                fem_mesh_plan** out) {
    if (!out) { set_error("fem_mesh_plan_create: out is NULL"); return FEM_ERR_INVALID_ARG; }
    *out = nullptr;
    if (dim != 2 && dim != 3) { set_error("fem_mesh_plan_create: dim must be 2 or 3 (got %d)", dim); return FEM_ERR_UNSUPPORTED; }
    if (n_elem < 0 || n_vert < 0) { set_error("fem_mesh_plan_create: negative size"); return FEM_ERR_INVALID_ARG; }
    if (n_elem > 0 && (n_vert == 0 || !conn)) {
        set_error("fem_mesh_plan_create: elements without vertices or NULL connectivity");
        return FEM_ERR_INVALID_ARG;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    fem_mesh_plan* p = new (std::nothrow) fem_mesh_plan();
    if (!p) { set_error("fem_mesh_plan_create: out of host memory"); return FEM_ERR_INVALID_ARG; }
    p->dim = dim;
    p->n_elem = n_elem;
    p->n_vert = n_vert;
    p->n_tiles = (n_elem + kPlanTile - 1) / kPlanTile;
    hipError_t e = hipGetDevice(&p->device);
    if (e == hipSuccess && n_elem > 0) {
        // tile_off, the totals and lidx share one allocation
        const size_t off_bytes = (size_t)(p->n_tiles + 1) * sizeof(int64_t);
        e = hipMalloc(&p->block, off_bytes + sizeof(MeshPlanTotals) + (size_t)n_elem * sizeof(uint32_t));
        MeshPlanTotals* totals = nullptr;
        if (e == hipSuccess) {
            char* base = static_cast<char*>(p->block);
            p->tile_off = reinterpret_cast<int64_t*>(base);
            totals = reinterpret_cast<MeshPlanTotals*>(base + off_bytes);
            p->lidx = reinterpret_cast<uint32_t*>(base + off_bytes + sizeof(MeshPlanTotals));
            e = dim == 2 ? launch_mesh_plan<3, false>(p, conn, s) : launch_mesh_plan<4, false>(p, conn, s);
        }
        if (e == hipSuccess) {
            hipLaunchKernelGGL(mesh_plan_scan_kernel, dim3(1), dim3(1024), 0, s, p->n_tiles, p->tile_off, totals);
            e = hipGetLastError();
        }
        MeshPlanTotals h{};
        if (e == hipSuccess) e = hipMemcpyAsync(&h, totals, sizeof h, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e == hipSuccess && h.bad) {
            mesh_plan_free(p);
            set_error("fem_mesh_plan_create: %lld vertex indices outside [0, %lld)", (long long)h.bad, (long long)n_vert);
            return FEM_ERR_INVALID_ARG;
        }
        p->total = h.total;
        p->max_tile = h.max_tile;
        if (e == hipSuccess) e = hipMalloc(&p->tile_verts, (size_t)h.total * sizeof(int32_t));
        if (e == hipSuccess) e = dim == 2 ? launch_mesh_plan<3, true>(p, conn, s) : launch_mesh_plan<4, true>(p, conn, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);   // any stream may use the plan from here on
    }
    if (e != hipSuccess) { mesh_plan_free(p); return hip_fail(e, "fem_mesh_plan_create"); }
    *out = p;
    return FEM_OK;
}

fem_status fem_mesh_plan_info(const fem_mesh_plan* plan, int* dim, int64_t* n_elem, int64_t* n_vert,
                              int* max_tile_vertices, int64_t* tile_vertices) {
    if (!plan) { set_error("fem_mesh_plan_info: NULL plan"); return FEM_ERR_INVALID_ARG; }
    if (dim) *dim = plan->dim;
    if (n_elem) *n_elem = plan->n_elem;
    if (n_vert) *n_vert = plan->n_vert;
    if (max_tile_vertices) *max_tile_vertices = plan->max_tile;
    if (tile_vertices) *tile_vertices = plan->total;
    return FEM_OK;
}

void fem_mesh_plan_destroy(fem_mesh_plan* plan) { mesh_plan_free(plan); }

fem_status fem_geometry_planned(const fem_mesh_plan* plan, const double* coords, int out_dtype, void* inv_j,
                               void* det_j, int32_t* counts, void* stream) {
    if (!plan) { set_error("fem_geometry_planned: NULL plan"); return FEM_ERR_INVALID_ARG; }
    if (out_dtype != FEM_F32 && out_dtype != FEM_F64) {
        set_error("fem_geometry_planned: unknown dtype %d", out_dtype);
        return FEM_ERR_UNSUPPORTED;
    }
    if (plan->n_elem == 0) return FEM_OK;
    if (!coords || !inv_j || !det_j) { set_error("fem_geometry_planned: NULL array"); return FEM_ERR_INVALID_ARG; }
    int dev = 0;
    if (hipGetDevice(&dev) == hipSuccess && dev != plan->device) {
        set_error("fem_geometry_planned: the plan was built on device %d, current device is %d", plan->device, dev);
        return FEM_ERR_INVALID_ARG;
    }
    const int maxc = std::max(plan->max_tile, 1);
    const size_t lds = (size_t)maxc * plan->dim * sizeof(double);
    const unsigned grid = (unsigned)std::min<int64_t>(std::max<int64_t>(plan->n_tiles, 1), (int64_t)1 << 30);
    hipStream_t s = static_cast<hipStream_t>(stream);
    auto go = [&](auto dim_c, auto out_c) {
        constexpr int D = decltype(dim_c)::value;
        using Out = typename decltype(out_c)::type;
        const bool whole = whole_lines(plan->n_elem, sizeof(Out), {inv_j, det_j});
        const auto k = whole ? geometry_planned_kernel<D, Out, true> : geometry_planned_kernel<D, Out, false>;
        hipLaunchKernelGGL(k, dim3(grid), dim3(64), lds, s, plan->n_elem, plan->n_tiles, plan->tile_off,
                           plan->tile_verts, plan->lidx, coords, static_cast<Out*>(inv_j), static_cast<Out*>(det_j),
                           counts, whole ? kOrderLaunch : kOrderXcd);
    };
    struct F32 { using type = float; };
    struct F64 { using type = double; };
    if (plan->dim == 2) {
        if (out_dtype == FEM_F32) go(std::integral_constant<int, 2>(), F32{});
        else go(std::integral_constant<int, 2>(), F64{});
    } else {
        if (out_dtype == FEM_F32) go(std::integral_constant<int, 3>(), F32{});
        else go(std::integral_constant<int, 3>(), F64{});
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_geometry_planned launch");
}

fem_status fem_integrate_residual_planned(const fem_mesh_plan* plan, int physics, int rule, int coef_space, int dtype,
                                          const double* coords, const void* u, const void* coef, void* elem_vec,
                                          void* inv_j, void* det_j, int32_t* counts, void* stream) {
    fem_status st = planned_common("fem_integrate_residual_planned", plan, physics, rule, coef_space, dtype, coords, u,
                                   coef, elem_vec, inv_j, det_j);
    if (st || plan->n_elem == 0) return st;
    const PlannedArgs a{plan, coords, u, coef, elem_vec, inv_j, det_j, counts, dtype, static_cast<hipStream_t>(stream)};
    const PlannedDispatch<false> f{a};
    hipError_t e = dispatch_element(plan->dim, physics, rule, coef_space, f, hipErrorInvalidValue);
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_integrate_residual_planned launch");
}

fem_status fem_integrate_residual_gather_planned(const fem_mesh_plan* plan, int physics, int rule, int coef_space,
                                                 int dtype, const double* coords, const void* u_vertex,
                                                 const void* coef, void* elem_vec, void* inv_j, void* det_j,
                                                 int32_t* counts, void* stream) {
    fem_status st = planned_common("fem_integrate_residual_gather_planned", plan, physics, rule, coef_space, dtype,
                                   coords, u_vertex, coef, elem_vec, inv_j, det_j);
    if (st || plan->n_elem == 0) return st;
    const PlannedArgs a{plan, coords, u_vertex, coef, elem_vec, inv_j, det_j, counts, dtype,
                        static_cast<hipStream_t>(stream)};
    const PlannedDispatch<true> f{a};
    hipError_t e = dispatch_element(plan->dim, physics, rule, coef_space, f, hipErrorInvalidValue);
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_integrate_residual_gather_planned launch");
}

}  // extern "C"
