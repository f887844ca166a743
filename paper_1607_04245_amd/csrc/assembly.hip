// assembly.hip -- the global residual from element vectors, and its adjoint.
//
// Section 2 writes the global residual as the sum over elements of each
// element vector mapped back through the element restriction (the transpose
// of the closure). Here that sum is a gather, not a scatter: a plan built
// once per mesh holds, for every vertex, the list of (element, local vertex)
// slots that touch it (the transpose of the connectivity, in compressed-row
// form), sorted by element. The assembly kernel gives each vertex one lane
// that adds its slots' entries in that order, starting from zero, so the
// result is deterministic (no atomics) and is exactly the element-by-element
// sum in increasing element order, evaluated in the working precision.
//
// The rows are stored sliced: for each group of 64 consecutive vertices (one
// wave), slot j of all 64 rows is contiguous, and every row of the group is
// padded with an empty marker to the group's longest row. A wave's j-th slot
// load is then one contiguous 256-byte access instead of 64 accesses one row
// apart; each vertex sees its own slots in element order.
//
// The plan is built on the device. Integer atomics count the slots of every
// vertex, find indices outside [0, n_vert) and hand every slot a place in its
// row; the places depend on timing, so after the slots are stored a wave per
// group sorts its 64 rows: it holds them in LDS and each entry counts the
// smaller ones of its row. For 400,003 tets creating the plan takes 171 us
// (377 us with a radix sort of all slots and its scratch). Meshes with a
// vertex of more than kLdsRow elements take that sort (keyed by vertex, stable,
// so rows stay in element order): its cost does not grow with the row.
//
// The restriction (closure) kernel is the adjoint: one lane per element
// copies the vertex values of its d+1 vertices into the SoA closure rows.
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include <new>

#include "fem_device.hpp"
#include "fem_internal.hpp"

struct fem_assembly_plan {
    int dim = 0;
    int device = 0;
    int64_t n_elem = 0;
    int64_t n_vert = 0;
    int64_t n_groups = 0;          // ceil(n_vert / 64)
    void* block = nullptr;         // the allocation that holds grp_off and grp_width
    int64_t* grp_off = nullptr;    // [n_groups + 1], first entry of each group in `sell`
    int32_t* grp_width = nullptr;  // [n_groups], slots per row in the group (its longest row)
    uint32_t* sell = nullptr;      // [grp_off[n_groups]]: group g, slot j, lane l at grp_off[g] + 64 j + l;
                                   // slot = e * (dim + 1) + b, or kNoSlot past the row's end
};

namespace femq {

constexpr uint32_t kNoSlot = 0xFFFFFFFFu;

// Rows up to this length are sorted in LDS: 64 rows of 256 slots fill 64 KB.
constexpr int kLdsRow = 256;

struct AssemblyTotals {
    int64_t entries;   // of sell
    int32_t widest;    // longest row
    int32_t bad;       // indices outside [0, n_vert)
};

// Slots per vertex, each slot's place in its row, and bad indices.
__global__ void __launch_bounds__(256)
assembly_count_kernel(int64_t m, int64_t n_vert, const int32_t* __restrict__ conn, int32_t* __restrict__ count,
                      uint32_t* __restrict__ place, int32_t* __restrict__ bad) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int nbad = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        const int32_t v = conn[i];
        if (v >= 0 && (int64_t)v < n_vert)
            place[i] = (uint32_t)atomicAdd(count + v, 1);
        else
            ++nbad;
    }
    if (nbad) atomicAdd(bad, nbad);
}

// Group widths: the longest row among each group's 64 vertices (vertices
// past n_vert count as empty rows). One wave per group.
__global__ void __launch_bounds__(256)
assembly_width_kernel(int64_t n_groups, int64_t n_vert, const int32_t* __restrict__ count, int32_t* __restrict__ width) {
    const int lane = threadIdx.x & 63;
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t g = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); g < n_groups; g += waves) {
        const int64_t v = g * 64 + lane;
        int32_t w = v < n_vert ? count[v] : 0;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) w = max(w, __shfl_xor(w, off, 64));
        if (lane == 0) width[g] = w;
    }
}

// First entry of every group (off[n_groups] = all entries) and the longest
// row. One workgroup walks the groups: 64 vertices each, so its 4096 widths
// per step are 2^18 vertices.
__global__ void __launch_bounds__(1024)
assembly_scan_kernel(int64_t n_groups, const int32_t* __restrict__ width, int64_t* __restrict__ off,
                     AssemblyTotals* __restrict__ totals) {
    __shared__ int64_t wave_sum[16];
    __shared__ int32_t wave_max[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t run = 0;
    int32_t most = 0;
    for (int64_t g0 = 0; g0 < n_groups; g0 += 4096) {
        const int64_t g = g0 + 4 * (int64_t)threadIdx.x;
        int64_t c[4], own = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int32_t w = g + r < n_groups ? width[g + r] : 0;
            most = max(most, w);
            c[r] = (int64_t)w * 64;
            own += c[r];
        }
        int64_t scan = own;   // inclusive over the wave
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t x = __shfl_up(scan, o, 64);
            if (lane >= o) scan += x;
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
            if (g + r < n_groups) off[g + r] = at;
            at += c[r];
        }
        __syncthreads();   // wave_sum is read before the next step writes it
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o, 64));
    if (lane == 0) wave_max[wave] = most;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) most = max(most, wave_max[w]);
        off[n_groups] = run;
        totals->entries = run;
        totals->widest = most;
    }
}

// Every slot to its place in its vertex's row.
__global__ void __launch_bounds__(256)
assembly_fill_kernel(int64_t m, const int32_t* __restrict__ conn, const uint32_t* __restrict__ place,
                     const int64_t* __restrict__ off, uint32_t* __restrict__ sell) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        const int32_t v = conn[i];
        sell[off[v / 64] + (int64_t)place[i] * 64 + v % 64] = (uint32_t)i;
    }
}

// Sorts the rows of a group and pads them: one wave per group, its rows in
// LDS (slot j of lane l at 64 j + l). An entry's place is the number of smaller
// ones in its row. A lane sorts its own row, which takes it w * w / 4 steps for the
// group's longest row w. A few rows above 32 slots among short ones are sorted by
// the whole wave instead, one after the other, a step per slot: one vertex of 200
// elements in a mesh of 1000 tets, plan 402 us with each lane on its own, 125
// this way.
__global__ void __launch_bounds__(64)
assembly_sort_kernel(int64_t n_groups, int64_t n_vert, const int32_t* __restrict__ count,
                     const int32_t* __restrict__ width, const int64_t* __restrict__ off, uint32_t* __restrict__ sell) {
    constexpr int kNarrow = 32, PER = kLdsRow / 64;
    extern __shared__ uint32_t rows[];
    const int lane = threadIdx.x;
    for (int64_t g = blockIdx.x; g < n_groups; g += gridDim.x) {
        const int64_t v = g * 64 + lane;
        const int32_t w = width[g], len = v < n_vert ? count[v] : 0;
        uint32_t* dst = sell + off[g] + lane;
        for (int32_t j = 0; j < w; ++j) {
            rows[j * 64 + lane] = j < len ? dst[(int64_t)j * 64] : kNoSlot;
        }
        int32_t wide_slots = len > kNarrow ? len : 0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) wide_slots += __shfl_xor(wide_slots, o, 64);
        const bool shared = wide_slots > 0 && 4 * wide_slots + kNarrow * kNarrow < w * w;
        const int32_t longest = shared ? kNarrow : w, own = shared && len > kNarrow ? 0 : len;
        __syncthreads();
        // four entries at a time share the walk over the row
        for (int32_t j = 0; j < longest; j += 4) {
            uint32_t x[4];
            int32_t rank[4] = {0, 0, 0, 0};
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = j + r < longest ? rows[(j + r) * 64 + lane] : kNoSlot;
#pragma unroll 4
            for (int32_t i = 0; i < longest; ++i) {
                const uint32_t y = rows[i * 64 + lane];
#pragma unroll
                for (int r = 0; r < 4; ++r) rank[r] += (int32_t)(y < x[r]);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (j + r < own) dst[(int64_t)rank[r] * 64] = x[r];
        }
        for (uint64_t wide = shared ? __ballot(len > kNarrow) : 0; wide != 0; wide &= wide - 1) {
            const int l = __builtin_ctzll(wide);
            const int32_t n = __shfl(len, l, 64);
            uint32_t x[PER];
            int32_t rank[PER];
#pragma unroll
            for (int r = 0; r < PER; ++r) {
                x[r] = lane + 64 * r < n ? rows[(lane + 64 * r) * 64 + l] : kNoSlot;
                rank[r] = 0;
            }
#pragma unroll 8
            for (int32_t i = 0; i < n; ++i) {
                const uint32_t y = rows[i * 64 + l];
#pragma unroll
                for (int r = 0; r < PER; ++r) rank[r] += (int32_t)(y < x[r]);
            }
#pragma unroll
            for (int r = 0; r < PER; ++r)
                if (lane + 64 * r < n) dst[(int64_t)rank[r] * 64 + l - lane] = x[r];
        }
        for (int32_t j = len; j < w; ++j) dst[(int64_t)j * 64] = kNoSlot;
        __syncthreads();   // the rows are read before the next group's are loaded
    }
}

// The radix path: slot numbers to sort, and the sliced storage of its result,
// entry (g, j, l) = slot j of vertex 64 g + l, or kNoSlot.
__global__ void __launch_bounds__(256)
assembly_ids_kernel(int64_t m, uint32_t* __restrict__ ids) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) ids[i] = (uint32_t)i;
}

__global__ void __launch_bounds__(256)
assembly_slice_kernel(int64_t n_groups, int64_t n_vert, const int32_t* __restrict__ row_ptr,
                      const uint32_t* __restrict__ slots, const int32_t* __restrict__ width,
                      const int64_t* __restrict__ off, uint32_t* __restrict__ sell) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_groups * 64; i += stride) {
        const int64_t g = i / 64, v = i;
        const int l = (int)(i % 64);
        const int32_t s0 = v < n_vert ? row_ptr[v] : 0, len = v < n_vert ? row_ptr[v + 1] - s0 : 0;
        const int32_t w = width[g];
        uint32_t* dst = sell + off[g] + l;
        for (int32_t j = 0; j < w; ++j) dst[(int64_t)j * 64] = j < len ? slots[s0 + j] : kNoSlot;
    }
}

// One wave per group of 64 vertices and NW of its NC components, one lane per
// vertex: vertex_vec[v][c] = sum over the vertex's slots, in slot order, of
// elem_vec[b * NC + c][e]. The rows are walked in chunks of CH slots whose loads
// are all issued before the first add (empty entries read a valid slot and
// their adds are skipped), so a lane waits about once per chunk instead of once
// per slot; the adds stay in slot order.
//
// What bounds it is the L1 and L2 traffic of the element rows: a lane's words
// of one slot lie some elements from its neighbour's, so a load touches about
// 24 lines whose other words belong to other slots. Hence the loads go row by
// row (component outside, slots inside), 12 slots a chunk, and the workgroups
// are numbered XCD by XCD, so that the groups that share lines share an L2. 3D
// elasticity FP64, 1,000,003 tets (96 MB of element vectors, 15 us): 42.8 us
// slot by slot in chunks of 16 in launch order, 38.5 XCD by XCD, 36.0 row by
// row, 34.0 with chunks of 12 (8: 37.2, 24: 35.0).
template <int NB, int NC, int NW, typename Real>
__global__ void __launch_bounds__(256)
assemble_kernel(int64_t n_vert, int64_t n_elem, int64_t n_groups, const int64_t* __restrict__ grp_off,
                const int32_t* __restrict__ grp_width, const uint32_t* __restrict__ sell,
                const Real* __restrict__ R, Real* __restrict__ out) {
    // vertices of tetrahedral meshes lie in about 24 elements, of triangular
    // meshes in about 6
    constexpr int CH = NB == 4 ? (NC == 1 ? 24 : 12) : 8;
    // One component has few rows to gather from, and workgroups in launch order
    // suit every mesh: FP32, 2^20 tets 11.8 us XCD by XCD where rows lie 2^22
    // bytes apart, 9.2 this way (9.6 with 16 slots in flight); 3,000,001
    // triangles 18.6 and 17.6.
    constexpr int ORDER = NC == 1 ? kOrderLaunch : kOrderXcd;
    constexpr int PARTS = NC / NW;
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const int64_t n_waves = (int64_t)gridDim.x * wpb;
    for (int64_t k = __builtin_amdgcn_readfirstlane((int)(row_block(ORDER) * wpb + (threadIdx.x >> 6)));
         k < n_groups * PARTS; k += n_waves) {
        const int64_t g = k / PARTS;
        const int c0 = (int)(k - g * PARTS) * NW;
        Real acc[NW];
#pragma unroll
        for (int c = 0; c < NW; ++c) acc[c] = Real(0);
        const uint32_t* row = sell + grp_off[g] + lane;
        const int32_t w = grp_width[g];
        for (int32_t s = 0; s < w; s += CH) {
            uint32_t sl[CH], e[CH], b[CH];
#pragma unroll
            for (int j = 0; j < CH; ++j) sl[j] = s + j < w ? row[(int64_t)(s + j) * 64] : kNoSlot;
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const uint32_t sj = sl[j] != kNoSlot ? sl[j] : 0u;
                e[j] = sj / NB;
                b[j] = sj - e[j] * NB;
            }
            Real r[CH][NW];
#pragma unroll
            for (int c = 0; c < NW; ++c)
#pragma unroll
                for (int j = 0; j < CH; ++j) r[j][c] = R[(int64_t)(b[j] * NC + c0 + c) * n_elem + e[j]];
#pragma unroll
            for (int j = 0; j < CH; ++j)
#pragma unroll
                for (int c = 0; c < NW; ++c) acc[c] = sl[j] != kNoSlot ? acc[c] + r[j][c] : acc[c];
        }
        const int64_t v = g * 64 + lane;
        if (v < n_vert) {
#pragma unroll
            for (int c = 0; c < NW; ++c) out[v * NC + c0 + c] = acc[c];
        }
    }
}

// One lane per element: elem_vec[b * NC + c][e] = vertex_vec[conn[e][b]][c];
// an index outside [0, n_vert) gives NaN entries and reads nothing outside.
template <int NB, int NC, typename Real>
__global__ void __launch_bounds__(256)
restrict_kernel(int64_t n_elem, int64_t n_vert, const int32_t* __restrict__ conn, const Real* __restrict__ vert,
                Real* __restrict__ out) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int32_t hi = vertex_hi(n_vert);
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n_elem; e += stride) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int32_t v = conn[e * NB + b];
            const bool ok = (v >= 0) & ((int64_t)v < n_vert);
            const int64_t vi = (int64_t)min(max(v, 0), hi);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const Real x = vert[vi * NC + c];
                out[(int64_t)(b * NC + c) * n_elem + e] = ok ? x : Real(__builtin_nan(""));
            }
        }
    }
}

static int grid_for(int64_t items) {
    const int64_t cap = (int64_t)std::max(device_cus(), 1) * 32;
    return (int)std::max<int64_t>(1, std::min<int64_t>((items + 255) / 256, cap));
}

// Below 2048 groups (131,072 vertices) a wave per group leaves SIMDs with less
// than two waves, and each component gets a wave of its own: 3D elasticity FP64,
// 100,003 tets (290 groups) 9.2 us with all three in one wave, 5.8 with three; at
// 2,097,152 tets (6000 groups) 65 and 68 us.
constexpr int64_t kSplitGroups = 2048;

template <int NB, int NC, typename Real>
static hipError_t launch_assemble_t(const fem_assembly_plan* p, const void* R, void* out, hipStream_t s) {
    const bool split = NC > 1 && p->n_groups < kSplitGroups;
    const auto k = split ? assemble_kernel<NB, NC, 1, Real> : assemble_kernel<NB, NC, NC, Real>;
    hipLaunchKernelGGL(k, dim3(grid_for(p->n_groups * 64 * (split ? NC : 1))), dim3(256), 0, s, p->n_vert, p->n_elem,
                       p->n_groups, p->grp_off, p->grp_width, p->sell, static_cast<const Real*>(R), static_cast<Real*>(out));
    return hipGetLastError();
}

template <int NB, typename Real>
static hipError_t launch_assemble_nc(int nc, const fem_assembly_plan* p, const void* R, void* out, hipStream_t s) {
    switch (nc) {
    case 1: return launch_assemble_t<NB, 1, Real>(p, R, out, s);
    case 2: return launch_assemble_t<NB, 2, Real>(p, R, out, s);
    case 3: return launch_assemble_t<NB, 3, Real>(p, R, out, s);
    default: return hipErrorInvalidValue;
    }
}

template <int NB, typename Real>
static hipError_t launch_restrict_nc(int nc, int64_t n_elem, int64_t n_vert, const int32_t* conn, const void* vert,
                                     void* out, hipStream_t s) {
    const dim3 g(grid_for(n_elem)), b(256);
    const Real* v = static_cast<const Real*>(vert);
    Real* o = static_cast<Real*>(out);
    switch (nc) {
    case 1: hipLaunchKernelGGL((restrict_kernel<NB, 1, Real>), g, b, 0, s, n_elem, n_vert, conn, v, o); break;
    case 2: hipLaunchKernelGGL((restrict_kernel<NB, 2, Real>), g, b, 0, s, n_elem, n_vert, conn, v, o); break;
    case 3: hipLaunchKernelGGL((restrict_kernel<NB, 3, Real>), g, b, 0, s, n_elem, n_vert, conn, v, o); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Fills p->sell from a stable radix sort of the slot numbers keyed by vertex:
// the rows come out in slot, hence element, order at any length. `ids` is
// scratch for the slot numbers, count[n_vert] is zero.
static hipError_t slice_by_radix_sort(const fem_assembly_plan* p, const int32_t* conn, int64_t m, const int32_t* count,
                                      uint32_t* ids, hipStream_t s) {
    const int64_t nv = p->n_vert, ng = p->n_groups;
    const uint32_t* keys = reinterpret_cast<const uint32_t*>(conn);  // valid indices are non-negative
    int end_bit = 1;
    while (end_bit < 32 && ((int64_t)1 << end_bit) < nv) ++end_bit;
    int32_t* row_ptr = nullptr;
    uint32_t *keys_out = nullptr, *slots = nullptr;
    void* temp = nullptr;
    size_t scan_bytes = 0, sort_bytes = 0;
    hipError_t e = hipMalloc(&row_ptr, (size_t)(nv + 1) * sizeof(int32_t));
    if (e == hipSuccess) e = hipMalloc(&keys_out, (size_t)m * sizeof(uint32_t));
    if (e == hipSuccess) e = hipMalloc(&slots, (size_t)m * sizeof(uint32_t));
    if (e == hipSuccess) e = hipcub::DeviceScan::ExclusiveSum(nullptr, scan_bytes, count, row_ptr, (int)(nv + 1), s);
    if (e == hipSuccess)
        e = hipcub::DeviceRadixSort::SortPairs(nullptr, sort_bytes, keys, keys_out, ids, slots, (int)m, 0, end_bit, s);
    if (e == hipSuccess) e = hipMalloc(&temp, std::max(scan_bytes, sort_bytes) + 16);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(assembly_ids_kernel, dim3(grid_for(m)), dim3(256), 0, s, m, ids);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipcub::DeviceScan::ExclusiveSum(temp, scan_bytes, count, row_ptr, (int)(nv + 1), s);
    if (e == hipSuccess)
        e = hipcub::DeviceRadixSort::SortPairs(temp, sort_bytes, keys, keys_out, ids, slots, (int)m, 0, end_bit, s);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(assembly_slice_kernel, dim3(grid_for(ng * 64)), dim3(256), 0, s, ng, nv, row_ptr, slots,
                           p->grp_width, p->grp_off, p->sell);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);   // the scratch dies here
    for (void* q : {(void*)row_ptr, (void*)keys_out, (void*)slots, temp})
        if (q) (void)hipFree(q);
    return e;
}

static void plan_free(fem_assembly_plan* p) {
    if (!p) return;
    if (p->block) (void)hipFree(p->block);
    if (p->sell) (void)hipFree(p->sell);
    delete p;
}

}  // namespace femq

using namespace femq;

extern "C" {

fem_status fem_assembly_plan_create(int dim, int64_t n_elem, int64_t n_vert, const int32_t* conn, void* stream,
                                    fem_assembly_plan** out) {
    if (!out) { set_error("fem_assembly_plan_create: out is NULL"); return FEM_ERR_INVALID_ARG; }
    *out = nullptr;
    if (dim != 2 && dim != 3) { set_error("fem_assembly_plan_create: dim must be 2 or 3 (got %d)", dim); return FEM_ERR_UNSUPPORTED; }
    if (n_elem < 0 || n_vert < 0) { set_error("fem_assembly_plan_create: negative size"); return FEM_ERR_INVALID_ARG; }
    if (n_elem > 0 && (n_vert == 0 || !conn)) {
        set_error("fem_assembly_plan_create: elements without vertices or NULL connectivity");
        return FEM_ERR_INVALID_ARG;
    }
    const int64_t m = n_elem * (dim + 1);
    if (m > (int64_t)INT32_MAX || n_vert >= (int64_t)INT32_MAX) {
        set_error("fem_assembly_plan_create: n_elem * (dim + 1) and n_vert must stay below 2^31");
        return FEM_ERR_UNSUPPORTED;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    fem_assembly_plan* p = new (std::nothrow) fem_assembly_plan();
    if (!p) { set_error("fem_assembly_plan_create: out of host memory"); return FEM_ERR_INVALID_ARG; }
    p->dim = dim;
    p->n_elem = n_elem;
    p->n_vert = n_vert;
    p->n_groups = (n_vert + 63) / 64;
    const int64_t ng = p->n_groups;
    // offsets, totals and widths share one allocation
    const size_t off_bytes = (size_t)(ng + 1) * sizeof(int64_t);
    hipError_t e = hipGetDevice(&p->device);
    if (e == hipSuccess) e = hipMalloc(&p->block, off_bytes + sizeof(AssemblyTotals) + (size_t)ng * sizeof(int32_t));
    if (e != hipSuccess) { plan_free(p); return hip_fail(e, "fem_assembly_plan_create: hipMalloc"); }
    p->grp_off = static_cast<int64_t*>(p->block);
    AssemblyTotals* totals = reinterpret_cast<AssemblyTotals*>(static_cast<char*>(p->block) + off_bytes);
    p->grp_width = reinterpret_cast<int32_t*>(totals + 1);
    if (m == 0) {  // no slots: every group has width 0
        e = hipMemsetAsync(p->block, 0, off_bytes + sizeof(AssemblyTotals) + (size_t)ng * sizeof(int32_t), s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) { plan_free(p); return hip_fail(e, "fem_assembly_plan_create"); }
        *out = p;
        return FEM_OK;
    }

    // scratch: slots per vertex, and every slot's place in its row
    int32_t* count = nullptr;
    e = hipMalloc(&count, (size_t)(n_vert + 1) * sizeof(int32_t) + (size_t)m * sizeof(uint32_t));
    if (e != hipSuccess) { plan_free(p); return hip_fail(e, "fem_assembly_plan_create: hipMalloc"); }
    uint32_t* place = reinterpret_cast<uint32_t*>(count + n_vert + 1);
    AssemblyTotals h{};
    e = hipMemsetAsync(count, 0, (size_t)(n_vert + 1) * sizeof(int32_t), s);
    if (e == hipSuccess) e = hipMemsetAsync(totals, 0, sizeof *totals, s);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(assembly_count_kernel, dim3(grid_for(m)), dim3(256), 0, s, m, n_vert, conn, count, place,
                           &totals->bad);
        hipLaunchKernelGGL(assembly_width_kernel, dim3(grid_for(ng * 64)), dim3(256), 0, s, ng, n_vert, count, p->grp_width);
        hipLaunchKernelGGL(assembly_scan_kernel, dim3(1), dim3(1024), 0, s, ng, p->grp_width, p->grp_off, totals);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(&h, totals, sizeof h, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e == hipSuccess && h.bad) {
        (void)hipFree(count);
        plan_free(p);
        set_error("fem_assembly_plan_create: %d vertex indices outside [0, %lld)", (int)h.bad, (long long)n_vert);
        return FEM_ERR_INVALID_ARG;
    }
    if (e == hipSuccess) e = hipMalloc(&p->sell, (size_t)std::max<int64_t>(h.entries, 1) * sizeof(uint32_t));
    if (e == hipSuccess && h.widest <= kLdsRow) {
        hipLaunchKernelGGL(assembly_fill_kernel, dim3(grid_for(m)), dim3(256), 0, s, m, conn, place, p->grp_off, p->sell);
        const int64_t grid = std::min<int64_t>(ng, (int64_t)1 << 22);
        hipLaunchKernelGGL(assembly_sort_kernel, dim3((unsigned)grid), dim3(64), (size_t)h.widest * 256, s, ng, n_vert, count,
                           p->grp_width, p->grp_off, p->sell);
        e = hipGetLastError();
    } else if (e == hipSuccess) {
        e = slice_by_radix_sort(p, conn, m, count, place, s);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFree(count);
    if (e != hipSuccess) { plan_free(p); return hip_fail(e, "fem_assembly_plan_create: index build"); }
    *out = p;
    return FEM_OK;
}

fem_status fem_assemble(const fem_assembly_plan* plan, int n_comp, int dtype, const void* elem_vec, void* vertex_vec,
                        void* stream) {
    if (!plan) { set_error("fem_assemble: NULL plan"); return FEM_ERR_INVALID_ARG; }
    if (n_comp < 1 || n_comp > 3) { set_error("fem_assemble: n_comp must be 1, 2 or 3 (got %d)", n_comp); return FEM_ERR_UNSUPPORTED; }
    if (dtype != FEM_F32 && dtype != FEM_F64) { set_error("fem_assemble: unknown dtype %d", dtype); return FEM_ERR_UNSUPPORTED; }
    if (plan->n_vert == 0) return FEM_OK;
    if (!vertex_vec || (plan->n_elem > 0 && !elem_vec)) { set_error("fem_assemble: NULL array"); return FEM_ERR_INVALID_ARG; }
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e;
    if (plan->dim == 2)
        e = dtype == FEM_F32 ? launch_assemble_nc<3, float>(n_comp, plan, elem_vec, vertex_vec, s)
                             : launch_assemble_nc<3, double>(n_comp, plan, elem_vec, vertex_vec, s);
    else
        e = dtype == FEM_F32 ? launch_assemble_nc<4, float>(n_comp, plan, elem_vec, vertex_vec, s)
                             : launch_assemble_nc<4, double>(n_comp, plan, elem_vec, vertex_vec, s);
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_assemble launch");
}

fem_status fem_assembly_plan_info(const fem_assembly_plan* plan, int* dim, int64_t* n_elem, int64_t* n_vert) {
    if (!plan) { set_error("fem_assembly_plan_info: NULL plan"); return FEM_ERR_INVALID_ARG; }
    if (dim) *dim = plan->dim;
    if (n_elem) *n_elem = plan->n_elem;
    if (n_vert) *n_vert = plan->n_vert;
    return FEM_OK;
}

void fem_assembly_plan_destroy(fem_assembly_plan* plan) { plan_free(plan); }

fem_status fem_restrict(int dim, int n_comp, int dtype, int64_t n_elem, int64_t n_vert, const int32_t* conn,
                        const void* vertex_vec, void* elem_vec, void* stream) {
    if (dim != 2 && dim != 3) { set_error("fem_restrict: dim must be 2 or 3 (got %d)", dim); return FEM_ERR_UNSUPPORTED; }
    if (n_comp < 1 || n_comp > 3) { set_error("fem_restrict: n_comp must be 1, 2 or 3 (got %d)", n_comp); return FEM_ERR_UNSUPPORTED; }
    if (dtype != FEM_F32 && dtype != FEM_F64) { set_error("fem_restrict: unknown dtype %d", dtype); return FEM_ERR_UNSUPPORTED; }
    if (n_elem < 0 || n_vert < 0) { set_error("fem_restrict: negative size"); return FEM_ERR_INVALID_ARG; }
    if (n_elem == 0) return FEM_OK;
    if (n_vert == 0) { set_error("fem_restrict: elements without vertices"); return FEM_ERR_INVALID_ARG; }
    if (!conn || !vertex_vec || !elem_vec) { set_error("fem_restrict: NULL array"); return FEM_ERR_INVALID_ARG; }
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e;
    if (dim == 2)
        e = dtype == FEM_F32 ? launch_restrict_nc<3, float>(n_comp, n_elem, n_vert, conn, vertex_vec, elem_vec, s)
                             : launch_restrict_nc<3, double>(n_comp, n_elem, n_vert, conn, vertex_vec, elem_vec, s);
    else
        e = dtype == FEM_F32 ? launch_restrict_nc<4, float>(n_comp, n_elem, n_vert, conn, vertex_vec, elem_vec, s)
                             : launch_restrict_nc<4, double>(n_comp, n_elem, n_vert, conn, vertex_vec, elem_vec, s);
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_restrict launch");
}

}  // extern "C"
