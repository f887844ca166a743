// fem_abi.hip -- the extern "C" entry points of libfemq (include/fem.h):
// argument validation, launch configuration, dispatch to the kernels.
//
// Validation happens before any HIP call, so invalid arguments are reported
// without touching a device. The hot-path calls never allocate, free or
// synchronize.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <tuple>

#include "fem.h"
#include "fem_internal.hpp"

namespace femq {

static thread_local std::string g_error;

void set_error(const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_error = buf;
}

fem_status hip_fail(hipError_t e, const char* what) {
    set_error("%s: %s (%d)", what, hipGetErrorString(e), (int)e);
    return FEM_ERR_HIP;
}

int device_cus() {
    static std::mutex mu;
    static int cache[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    std::lock_guard<std::mutex> lock(mu);
    if (cache[dev] == 0) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess) cache[dev] = cus;
    }
    return cache[dev];
}

// ------------------------------------------------------------- validation --

static bool valid_dim(int dim) { return dim == 2 || dim == 3; }
static bool valid_dtype(int dt) { return dt == FEM_F32 || dt == FEM_F64; }
static bool valid_phys(int p) { return p == FEM_LAPLACE || p == FEM_ELASTICITY || p == FEM_MASS; }
static bool valid_rule(int dim, int rule) {
    return rule == FEM_RULE_CENTROID || (dim == 2 && rule == FEM_RULE_TRI3) || (dim == 3 && rule == FEM_RULE_TET4);
}

static bool valid_space(int sp) { return sp == FEM_COEF_QUAD || sp == FEM_COEF_P1 || sp == FEM_COEF_P0; }

static fem_status check_space(const char* fn, int space) {
    if (!valid_space(space)) { set_error("%s: unknown coefficient space %d", fn, space); return FEM_ERR_UNSUPPORTED; }
    return FEM_OK;
}

// Rules of the second-order entry points: the degree-2 and degree-4 rules.
static bool valid_rule_p2(int dim, int rule) {
    return dim == 2 ? (rule == FEM_RULE_TRI3 || rule == FEM_RULE_TRI6) : (rule == FEM_RULE_TET4 || rule == FEM_RULE_TET11);
}

static fem_status check_combo_p2(const char* fn, int dim, int phys, int rule, int dtype) {
    if (!valid_dim(dim)) { set_error("%s: dim must be 2 or 3 (got %d)", fn, dim); return FEM_ERR_UNSUPPORTED; }
    if (!valid_phys(phys)) { set_error("%s: unknown physics %d", fn, phys); return FEM_ERR_UNSUPPORTED; }
    if (!valid_rule_p2(dim, rule)) { set_error("%s: rule %d is not available for P2 in %dD", fn, rule, dim); return FEM_ERR_UNSUPPORTED; }
    if (!valid_dtype(dtype)) { set_error("%s: unknown dtype %d", fn, dtype); return FEM_ERR_UNSUPPORTED; }
    return FEM_OK;
}

// P3 elements take the degree-4 rule of their dimension, which integrates
// a stiffness entry with a constant coefficient exactly.
static fem_status check_combo_p3(const char* fn, int dim, int phys, int rule, int dtype) {
    if (!valid_dim(dim)) { set_error("%s: dim must be 2 or 3 (got %d)", fn, dim); return FEM_ERR_UNSUPPORTED; }
    if (!valid_phys(phys)) { set_error("%s: unknown physics %d", fn, phys); return FEM_ERR_UNSUPPORTED; }
    if (rule != (dim == 2 ? FEM_RULE_TRI6 : FEM_RULE_TET11)) {
        set_error("%s: P3 in %dD takes rule %d only (got %d)", fn, dim, dim == 2 ? FEM_RULE_TRI6 : FEM_RULE_TET11, rule);
        return FEM_ERR_UNSUPPORTED;
    }
    if (!valid_dtype(dtype)) { set_error("%s: unknown dtype %d", fn, dtype); return FEM_ERR_UNSUPPORTED; }
    return FEM_OK;
}

// Rules of the element-matrix entry point for each order.
static bool valid_rule_jac(int dim, int order, int rule) {
    const int low = dim == 2 ? FEM_RULE_TRI3 : FEM_RULE_TET4, high = dim == 2 ? FEM_RULE_TRI6 : FEM_RULE_TET11;
    if (order == 3) return rule == high;
    return rule == low || (order == 1 && rule == FEM_RULE_CENTROID) || (order == 2 && rule == high);
}

static fem_status check_combo_jac(const char* fn, int dim, int phys, int order, int rule, int dtype) {
    if (!valid_dim(dim)) { set_error("%s: dim must be 2 or 3 (got %d)", fn, dim); return FEM_ERR_UNSUPPORTED; }
    if (!valid_phys(phys)) { set_error("%s: unknown physics %d", fn, phys); return FEM_ERR_UNSUPPORTED; }
    if (order < 1 || order > 3) { set_error("%s: order must be 1, 2 or 3 (got %d)", fn, order); return FEM_ERR_UNSUPPORTED; }
    if (!valid_rule_jac(dim, order, rule)) {
        set_error("%s: rule %d is not available for order %d in %dD", fn, rule, order, dim);
        return FEM_ERR_UNSUPPORTED;
    }
    if (!valid_dtype(dtype)) { set_error("%s: unknown dtype %d", fn, dtype); return FEM_ERR_UNSUPPORTED; }
    return FEM_OK;
}

static fem_status check_combo(const char* fn, int dim, int phys, int rule, int dtype) {
    if (!valid_dim(dim)) { set_error("%s: dim must be 2 or 3 (got %d)", fn, dim); return FEM_ERR_UNSUPPORTED; }
    if (!valid_phys(phys)) { set_error("%s: unknown physics %d", fn, phys); return FEM_ERR_UNSUPPORTED; }
    if (!valid_rule(dim, rule)) { set_error("%s: rule %d is not defined in %dD", fn, rule, dim); return FEM_ERR_UNSUPPORTED; }
    if (!valid_dtype(dtype)) { set_error("%s: unknown dtype %d", fn, dtype); return FEM_ERR_UNSUPPORTED; }
    return FEM_OK;
}

// ---------------------------------------------------------------- tuning --

typedef std::tuple<int, int, int, int, int> TuneKey;
static std::mutex g_tune_mu;
static std::map<TuneKey, fem_tuning> g_tune;

static bool valid_op(int op) {
    return op == FEM_OP_RESIDUAL || op == FEM_OP_RESIDUAL_MESH || op == FEM_OP_GEOMETRY || op == FEM_OP_BACKWARD ||
           op == FEM_OP_RESIDUAL_GATHER || op == FEM_OP_RESIDUAL_P2 || op == FEM_OP_BACKWARD_P2 ||
           op == FEM_OP_JACOBIAN || op == FEM_OP_JACOBIAN_P2 || op == FEM_OP_RESIDUAL_P3 || op == FEM_OP_BACKWARD_P3 ||
           op == FEM_OP_JACOBIAN_P3;
}

// Ops whose kernels take one element per lane and at most four waves per
// workgroup (register-heavy elements).
static bool one_per_lane_op(int op) {
    return op == FEM_OP_RESIDUAL_P2 || op == FEM_OP_BACKWARD_P2 || op == FEM_OP_JACOBIAN || op == FEM_OP_JACOBIAN_P2 ||
           op == FEM_OP_RESIDUAL_P3 || op == FEM_OP_BACKWARD_P3 || op == FEM_OP_JACOBIAN_P3;
}

// The geometry does not depend on physics or rule: one key per (dim, dtype).
static TuneKey tune_key(int op, int dim, int phys, int rule, int dtype) {
    if (op == FEM_OP_GEOMETRY) phys = rule = 0;
    return TuneKey(op, dim, phys, rule, dtype);
}

// Built-in launch configurations: the winners of the autotuner's sweep on
// one MI355X for the benchmark workloads; other combinations use the robust
// middle choice. Where none was set or tuned, p1_tuning and the element
// matrices refine them by count and alignment.
static fem_tuning default_tuning(int op, int dim, int phys, int rule, int dtype) {
    const bool f32 = dtype == FEM_F32;
    // RESIDUAL, BACKWARD (whole lines; p1_tuning has odd words): four waves in FP32
    // (two: 2 % slower at 100 to 460 MB), two in FP64 (four: 2D 2 % slower at 540 MB),
    // one for scalar forms on FP64 tets (230 MB: 37.8 us, 41.0 with two)
    const fem_tuning t{FEM_STRATEGY_LANE, 1, f32 ? 4 : dim == 3 && phys != FEM_ELASTICITY ? 1 : 2, 0};
    if (op == FEM_OP_GEOMETRY) return fem_tuning{FEM_STRATEGY_LANE, 4, 4, 0};
    // Store-bound. FP64 scalar matrices stream best with one wave (P2 3D Laplacian,
    // 30,720 tets 9.4 us, 10.5 with four; P1 245,760 tets 12.0, 13.1 with two), the
    // larger P2 elements with four (3D elasticity FP64, 40,960 tets 80 us, 84 with one;
    // 3D Laplacian FP32, 491,520 tets 55 and 59).
    if (op == FEM_OP_JACOBIAN_P2) return fem_tuning{FEM_STRATEGY_LANE, 1, f32 || phys == FEM_ELASTICITY ? 4 : 1, phys == FEM_ELASTICITY ? 16 : 0};
    if (op == FEM_OP_JACOBIAN) return fem_tuning{FEM_STRATEGY_LANE, 1, f32 && phys != FEM_ELASTICITY ? 2 : 1, 0};
    // P3: the 3D elements hold 20-60 closure and output words per lane, and
    // single-wave workgroups measured fastest there; 2D streams better with
    // four. (The component split of 3D elasticity, 2^21 tets: FP32 280 us, the
    // lane kernel 242; FP64 584 and 485.)
    if (op == FEM_OP_RESIDUAL_P3 || op == FEM_OP_BACKWARD_P3) return fem_tuning{FEM_STRATEGY_LANE, 1, dim == 3 ? 1 : 4, 0};
    if (op == FEM_OP_JACOBIAN_P3) return fem_tuning{FEM_STRATEGY_LANE, 1, 4, 0};
    // P2 (the remaining ops of one element per lane): four waves (2D elasticity FP32,
    // 2^22 triangles: 116 us with two, 110 with four; 2D FP64 at odd words, 620 MB: 4 %
    // slower with two), one for FP64 tets (3D elasticity adjoint, 1,000,001 tets: 270,
    // 287 with two; residuals and adjoints at 300 MB 8 % slower with four).
    if (one_per_lane_op(op)) return fem_tuning{FEM_STRATEGY_LANE, 1, f32 || dim == 2 ? 4 : 1, 0};
    if (op == FEM_OP_RESIDUAL_GATHER) return fem_tuning{FEM_STRATEGY_LANE, 2, 1, 0};
    if (op == FEM_OP_RESIDUAL_MESH) {
        if (phys == FEM_LAPLACE && f32) return fem_tuning{FEM_STRATEGY_LANE, 1, 1, 8};
        if (phys == FEM_ELASTICITY && f32) return fem_tuning{FEM_STRATEGY_LANE, 2, 2, 0};
        return fem_tuning{FEM_STRATEGY_LANE, 2, 1, 0};
    }
    return t;
}

// The matrix-core transposition exists for P3 tetrahedra with an f1 physics.
static bool mfma_available(int op, int dim, int phys) {
    return op == FEM_OP_RESIDUAL_P3 && dim == 3 && (phys == FEM_LAPLACE || phys == FEM_ELASTICITY);
}

// The component-parallel kernel exists for P3 tetrahedra with elasticity.
static bool component_available(int op, int dim, int phys) {
    return op == FEM_OP_RESIDUAL_P3 && dim == 3 && phys == FEM_ELASTICITY;
}

static bool valid_tuning(int op, const fem_tuning& t) {
    const bool strategy_ok = t.strategy == FEM_STRATEGY_LANE ||
                             ((t.strategy == FEM_STRATEGY_TRANSPOSE || t.strategy == FEM_STRATEGY_SHUFFLE) &&
                              op == FEM_OP_RESIDUAL) ||
                             ((t.strategy == FEM_STRATEGY_MFMA || t.strategy == FEM_STRATEGY_COMPONENT) &&
                              op == FEM_OP_RESIDUAL_P3) ||
                             (t.strategy == FEM_STRATEGY_DEDUP && op == FEM_OP_RESIDUAL_MESH && t.vec == 1);
    const bool one = one_per_lane_op(op);
    const bool vec_ok = one ? t.vec == 1 : (t.vec == 1 || t.vec == 2 || t.vec == 4);
    const bool waves_ok = t.waves_per_block == 1 || t.waves_per_block == 2 || t.waves_per_block == 4 ||
                          (t.waves_per_block == 8 && !one);
    return strategy_ok && vec_ok && waves_ok &&
           t.blocks_per_cu >= 0 && t.blocks_per_cu <= 64;
}

// The tuning cache named by the FEM_TUNE_CACHE environment variable is loaded
// once, before the first lookup or change of a tuning, so that explicit
// settings made afterwards take precedence. A missing file, or one without
// entries for this device, leaves the defaults (and the caller's error
// message) untouched. Lookups from other threads while the file is being
// read see the defaults.
static std::atomic<int> g_env_cache{0};   // 0 not loaded, 1 loading, 2 done

static void load_env_cache() {
    if (g_env_cache.load(std::memory_order_acquire) == 2) return;
    int expected = 0;
    if (!g_env_cache.compare_exchange_strong(expected, 1)) return;   // loaded or being loaded
    const char* path = std::getenv("FEM_TUNE_CACHE");
    if (path && *path) {
        const std::string saved = g_error;
        (void)fem_load_tuning(path);   // its fem_set_tuning calls return here at once
        g_error = saved;
    }
    g_env_cache.store(2, std::memory_order_release);
}

fem_tuning get_tuning(int op, int dim, int phys, int rule, int dtype, bool* chosen) {
    load_env_cache();
    std::lock_guard<std::mutex> lock(g_tune_mu);
    auto it = g_tune.find(tune_key(op, dim, phys, rule, dtype));
    if (chosen) *chosen = it != g_tune.end();
    return it != g_tune.end() ? it->second : default_tuning(op, dim, phys, rule, dtype);
}

void drop_tuning(int op, int dim, int phys, int rule, int dtype) {
    std::lock_guard<std::mutex> lock(g_tune_mu);
    g_tune.erase(tune_key(op, dim, phys, rule, dtype));
}

void put_tuning(int op, int dim, int phys, int rule, int dtype, const fem_tuning& t) {
    load_env_cache();
    std::lock_guard<std::mutex> lock(g_tune_mu);
    g_tune[tune_key(op, dim, phys, rule, dtype)] = t;
}

// Words per element that an order-k residual reads and writes as rows: the
// geometry, n_closure closures (u, w, R, du) and n_coef coefficient sets.
static int64_t row_words(int dim, int phys, int rule, int space, int order, int n_closure, int n_coef_sets) {
    const int nb = order == 1 ? dim + 1 : order == 2 ? (dim + 1) * (dim + 2) / 2 : (dim == 2 ? 10 : 20);
    const int nc = phys == FEM_ELASTICITY ? dim : 1, m = phys == FEM_ELASTICITY ? 2 : 1;
    const int nq = rule == FEM_RULE_CENTROID ? 1 : rule == FEM_RULE_TRI6 ? 6 : rule == FEM_RULE_TET11 ? 11 : dim + 1;
    const int nw = space == FEM_COEF_QUAD ? nq : space == FEM_COEF_P1 ? dim + 1 : 1;
    return dim * dim + 1 + (int64_t)n_closure * nb * nc + (int64_t)n_coef_sets * m * nw;
}

// Stores and workgroup order of a launch over rows of order-k elements, pitch bytes apart;
// whole: every output row starts on a 128-byte line. Runs: 16 consecutive workgroups
// per XCD. One MI355X, inputs rotating through more than the last-level cache holds;
// times relative to streaming stores in launch order unless said otherwise, means
// over the Laplacian and elasticity, residual and adjoint.
//  - Rows at odd words: plain stores in runs, so that the two parts of a line at a
//    wave's edge meet in the L2 that neighbouring workgroups share: P1 FP32 0.82 at
//    100 MB, 0.73 at 300, P2 FP32 0.72 and 0.67. (XCD by XCD 0.81 and 0.77 for P1, 1 %
//    faster up to 100 MB, 2 to 7 % slower from 400 on, except on P3 tets: FP32, 200
//    MB 0.63 and in runs 0.64, 900 MB 0.76 and 0.79. P2 below 384 MiB goes XCD by XCD
//    too: runs are 2 % faster over 60 to 380 MB, but not evenly, and 230 MB is 4 to 8 %
//    slower: 3D Laplacian FP64, 700,001 tets 43.4 us, 40.3 XCD by XCD.) P1 on FP64
//    triangles, where a wave's row has but two shared lines in five, streams from 544
//    MiB on (750 MB: 0.96 of the first version's time, in runs 1.00; FP64 tets 0.80 and
//    0.79).
//  - Whole lines that the 256 MB last-level cache can hold in part: plain stores in
//    runs. Residuals: P1 0.97 at 130 to 300 MB, 0.99 at 450, 1.04 at 540; P2 0.97, 0.99
//    (3D elasticity 1.08) and 1.05; P3 0.98, 1.05 and 1.07. Adjoints: P1 0.97, 0.95 and
//    1.05, P2 0.97, 1.03 and 1.07, P3 0.97, 0.98 and 1.09. XCD by XCD, each XCD writing
//    its own eighth of every row, is 3 % slower at 400 MB.
//  - Whole lines above those limits, and below 64 MiB on P2 and 128 on P3 tets, where
//    plain stores push the inputs out (P3 tets, 60 MB: FP32 0.85 of the first version's
//    time streamed, 0.91 plain; FP64 0.78 and 0.86; P2 3D elasticity, 40 MB, 16 % faster
//    streamed; triangles at 10 to 66 MB 3 % slower): streaming stores in launch order.
//    XCD by XCD they are 7 % slower at 700 MB.
//  - `stream` asks for that at any size, where plain stores gain nothing: P3
//    elasticity residuals on tets and on FP64 triangles, whose 20 or 60 rows leave in
//    one burst after a long element (3D FP64, 230 MB: 33 us and 37; 2D: 43 and 48; FP32
//    triangles 170 MB 32.0 and 29.7), and P1 residuals of scalar forms on FP64 tets, 4
//    rows out of 22 (230 MB: 37.8 and 39.0 us).
//  - Rows a multiple of 8 MiB apart (P3: 4), as with a power of two of elements, meet in
//    the same memory channels; there the XCDs stay apart, each in its own eighth of the
//    rows, streaming from 512 MiB on. 2D elasticity FP32, 2^22 triangles (386 MB) 65.6 us
//    in runs, 59.8 XCD by XCD; 3D Laplacian FP64, 2^21 tets (369 MB) 71 streaming, 56; 3D
//    elasticity FP64 (705 MB) 126 streaming in launch order, 112 XCD by XCD. P3 residuals
//    on tets stream from 448 MiB on (Laplacian FP64, 2^20 tets, 107 us plain, 101). An
//    odd multiple of 2 MiB: the rules above.
static void set_rows(Launch& l, bool whole, int dim, int dtype, int64_t pitch, int64_t rows, int order, bool adjoint,
                     bool stream = false) {
    const int64_t mib = pitch * rows >> 20;
    if (whole && pitch % ((int64_t)(order == 3 ? 4 : 8) << 20) == 0) {
        l.stream_out = mib >= (order == 3 && dim == 3 && !adjoint ? 448 : 512);
        l.order = order < 3 || mib >= 192 ? kOrderXcd : kOrderRuns;
        return;
    }
    const int64_t low = order == 1 || dim == 2 ? 0 : order == 3 ? 128 : 64;
    const int64_t high = !adjoint && (order == 1 || dim == 2) ? 448 : 416;
    const bool xcd = !whole && (order == 2 ? mib < 384 : order == 3 && dim == 3);
    if (order == 1 && pitch % ((int64_t)4 << 20) == 0) stream = false;   // 524,288 tets 18.8 us, 16.8 plain
    l.stream_out = whole ? stream || mib < low || mib >= high : order == 1 && dim == 2 && dtype == FEM_F64 && mib >= 544;
    l.order = l.stream_out ? kOrderLaunch : xcd ? kOrderXcd : kOrderRuns;
}

// Built-in configuration of the P1 lane kernels for n elements, `bytes` of rows.
//  - Whole lines: the default; rows a multiple of 4 MiB apart take four waves in FP64
//    too (2^21 tets, 3D Laplacian 61.5 us with one, 56.3 with four, adjoint 82.1, 77.3).
//  - Rows at odd words, but on 16 bytes (even: a count and arrays that allow it): 16
//    bytes per lane and one wave, so that a wave shares 2 of its 9 lines with its
//    neighbours and not 2 of 3, where that leaves five waves per CU and the rows are
//    more than the caches of the XCDs hold: FP32, 3D Laplacian, 500,004 tets 8.7 us, 9.1
//    with one element per lane, adjoint 11.2 and 12.6, 2,840,580 tets 43.1 and 45.1; FP64,
//    2D elasticity, 420,868 triangles 12.2 and 12.7; but FP32 2D Laplacian, 500,004
//    triangles (28 MB) 7.1 and 6.4.
//  - Off 16 bytes each such access is split: only from six waves per SIMD on in FP32
//    (2,272,267 tets 36.8 us with one element per lane, 35.0 with four; but the adjoint on
//    735,243 tets 17.6 and 19.5; FP64 the same), else one element and four waves.
static fem_tuning p1_tuning(const fem_tuning& t, int dtype, int64_t n, int64_t bytes, bool whole, bool even) {
    const int word = dtype == FEM_F32 ? 4 : 8, vec = 16 / word;
    const fem_tuning one{FEM_STRATEGY_LANE, 1, 4, 0}, wide{FEM_STRATEGY_LANE, vec, 1, 0};
    if (whole) return n * word % ((int64_t)4 << 20) == 0 ? one : t;
    if (even) return n >= (int64_t)vec * 64 * 1280 && bytes >= (int64_t)32 << 20 ? wide : one;
    return dtype == FEM_F32 && n >= (int64_t)vec * 64 * 6144 ? wide : one;
}

static Launch make_launch(const fem_tuning& t, int64_t work_items, int vec, hipStream_t s) {
    Launch l;
    l.vec = vec;
    l.block = 64 * t.waves_per_block;
    l.stream = s;
    l.max_grid = 1 << 22;  // the grid-stride loop covers the rest
    if (t.blocks_per_cu > 0) {
        int cus = device_cus();
        l.max_grid = std::min(l.max_grid, t.blocks_per_cu * (cus > 0 ? cus : 256));
    }
    l.grid = grid_for_lanes(l, work_items);
    return l;
}

// Kernels that give each wave tiles of 64*ept elements.
static Launch make_tile_launch(const fem_tuning& t, int64_t n, hipStream_t s) {
    const int64_t tiles = (n + 64 * t.vec - 1) / (64 * t.vec);
    Launch l = make_launch(t, tiles * 64, t.vec, s);
    return l;
}

static fem_status check_tuning_args(const char* fn, int op, int dim, int physics, int rule, int dtype) {
    if (!valid_op(op)) { set_error("%s: unknown op %d", fn, op); return FEM_ERR_UNSUPPORTED; }
    if (op == FEM_OP_GEOMETRY) {
        if (!valid_dim(dim)) { set_error("%s: dim must be 2 or 3 (got %d)", fn, dim); return FEM_ERR_UNSUPPORTED; }
        if (!valid_dtype(dtype)) { set_error("%s: unknown dtype %d", fn, dtype); return FEM_ERR_UNSUPPORTED; }
        return FEM_OK;
    }
    if (op == FEM_OP_RESIDUAL_P2 || op == FEM_OP_BACKWARD_P2) return check_combo_p2(fn, dim, physics, rule, dtype);
    if (op == FEM_OP_RESIDUAL_P3 || op == FEM_OP_BACKWARD_P3) return check_combo_p3(fn, dim, physics, rule, dtype);
    if (op == FEM_OP_JACOBIAN || op == FEM_OP_JACOBIAN_P2)
        return check_combo_jac(fn, dim, physics, op == FEM_OP_JACOBIAN ? 1 : 2, rule, dtype);
    if (op == FEM_OP_JACOBIAN_P3) return check_combo_jac(fn, dim, physics, 3, rule, dtype);
    return check_combo(fn, dim, physics, rule, dtype);
}

}  // namespace femq

using namespace femq;

extern "C" {

const char* fem_last_error(void) { return g_error.c_str(); }

fem_status fem_get_tuning(int op, int dim, int physics, int rule, int dtype, fem_tuning* out) {
    fem_status st = check_tuning_args("fem_get_tuning", op, dim, physics, rule, dtype);
    if (st) return st;
    if (!out) { set_error("fem_get_tuning: out is NULL"); return FEM_ERR_INVALID_ARG; }
    *out = get_tuning(op, dim, physics, rule, dtype);
    return FEM_OK;
}

fem_status fem_set_tuning(int op, int dim, int physics, int rule, int dtype, const fem_tuning* t) {
    fem_status st = check_tuning_args("fem_set_tuning", op, dim, physics, rule, dtype);
    if (st) return st;
    if (!t || !valid_tuning(op, *t)) { set_error("fem_set_tuning: invalid tuning for op %d", op); return FEM_ERR_INVALID_ARG; }
    if (t->strategy == FEM_STRATEGY_SHUFFLE && physics == FEM_ELASTICITY) {
        set_error("fem_set_tuning: the quad-permutation strategy covers scalar fields (Laplacian, mass)");
        return FEM_ERR_UNSUPPORTED;
    }
    if (t->strategy == FEM_STRATEGY_DEDUP && t->waves_per_block != 2 && t->waves_per_block != 4) {
        set_error("fem_set_tuning: the deduplicating strategy runs two or four waves per workgroup");
        return FEM_ERR_UNSUPPORTED;
    }
    if (t->strategy == FEM_STRATEGY_MFMA && !mfma_available(op, dim, physics)) {
        set_error("fem_set_tuning: the matrix-core strategy covers P3 tetrahedra with the Laplacian or elasticity");
        return FEM_ERR_UNSUPPORTED;
    }
    if (t->strategy == FEM_STRATEGY_COMPONENT && !component_available(op, dim, physics)) {
        set_error("fem_set_tuning: the component-parallel strategy covers P3 tetrahedra with elasticity");
        return FEM_ERR_UNSUPPORTED;
    }
    if (t->strategy == FEM_STRATEGY_COMPONENT && t->waves_per_block > comp_max_groups(dtype)) {
        set_error("fem_set_tuning: the component-parallel strategy runs at most %d three-wave group(s) per workgroup "
                  "for this dtype", comp_max_groups(dtype));
        return FEM_ERR_UNSUPPORTED;
    }
    put_tuning(op, dim, physics, rule, dtype, *t);
    return FEM_OK;
}

fem_status fem_geometry(int dim, int64_t n_elem, int64_t n_vert, const double* coords, const int32_t* conn,
                        int out_dtype, void* inv_j, void* det_j, int32_t* counts, void* stream) {
    if (!valid_dim(dim)) { set_error("fem_geometry: dim must be 2 or 3 (got %d)", dim); return FEM_ERR_INVALID_ARG; }
    if (!valid_dtype(out_dtype)) { set_error("fem_geometry: unknown dtype %d", out_dtype); return FEM_ERR_UNSUPPORTED; }
    if (n_elem < 0 || n_vert < 0) { set_error("fem_geometry: negative size"); return FEM_ERR_INVALID_ARG; }
    if (n_elem == 0) return FEM_OK;
    if (n_vert == 0) { set_error("fem_geometry: elements without vertices"); return FEM_ERR_INVALID_ARG; }
    if (!coords || !conn || !inv_j || !det_j) { set_error("fem_geometry: NULL array"); return FEM_ERR_INVALID_ARG; }
    const fem_tuning t = get_tuning(FEM_OP_GEOMETRY, dim, 0, 0, out_dtype);
    Launch l = make_tile_launch(t, n_elem, static_cast<hipStream_t>(stream));
    l.stream_out = whole_lines(n_elem, out_dtype == FEM_F32 ? 4 : 8, {inv_j, det_j});
    hipError_t e = launch_geometry(dim, out_dtype, n_elem, n_vert, coords, conn, inv_j, det_j, counts, l);
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_geometry launch");
}

fem_status fem_integrate_residual(int dim, int physics, int rule, int coef_space, int dtype, int64_t n_elem,
                                  const void* inv_j, const void* det_j, const void* u, const void* coef, void* elem_vec,
                                  void* stream) {
    fem_status st = check_combo("fem_integrate_residual", dim, physics, rule, dtype);
    if (!st) st = check_space("fem_integrate_residual", coef_space);
    if (st) return st;
    if (n_elem < 0) { set_error("fem_integrate_residual: negative n_elem"); return FEM_ERR_INVALID_ARG; }
    if (n_elem == 0) return FEM_OK;
    if (!inv_j || !det_j || !u || !coef || !elem_vec) {
        set_error("fem_integrate_residual: NULL array");
        return FEM_ERR_INVALID_ARG;
    }
    bool chosen;
    fem_tuning t = get_tuning(FEM_OP_RESIDUAL, dim, physics, rule, dtype, &chosen);
    ResidualArgs a{n_elem, inv_j, det_j, u, coef, elem_vec};
    hipError_t e;
    if (t.strategy == FEM_STRATEGY_TRANSPOSE) {
        int threads = transpose_block_threads(dim, physics, rule, coef_space, dtype, t.waves_per_block);
        if (threads == 0) { set_error("fem_integrate_residual: transpose strategy unavailable"); return FEM_ERR_UNSUPPORTED; }
        Launch l = make_launch(t, n_elem, 1, static_cast<hipStream_t>(stream));
        l.block = threads;
        e = launch_residual_transpose(dim, physics, rule, coef_space, dtype, a, l);
    } else if (t.strategy == FEM_STRATEGY_SHUFFLE) {
        if (physics == FEM_ELASTICITY) {
            set_error("fem_integrate_residual: the quad-permutation strategy covers scalar fields");
            return FEM_ERR_UNSUPPORTED;
        }
        Launch l = make_launch(t, (n_elem + 15) / 16 * 64, 1, static_cast<hipStream_t>(stream));
        e = launch_residual_shuffle(dim, physics, rule, coef_space, dtype, a, l);
    } else {
        const size_t word = dtype == FEM_F32 ? 4 : 8;
        const bool whole = whole_lines(n_elem, word, {elem_vec});
        const int64_t pitch = n_elem * (int64_t)word, rows = row_words(dim, physics, rule, coef_space, 1, 2, 1);
        if (!chosen) t = p1_tuning(t, dtype, n_elem, pitch * rows, whole,
                                   whole_lines(n_elem, word, {inv_j, det_j, u, coef, elem_vec}, 16));
        Launch l = make_launch(t, (n_elem + t.vec - 1) / t.vec, t.vec, static_cast<hipStream_t>(stream));
        set_rows(l, whole, dim, dtype, pitch, rows, 1, false,
                 dim == 3 && dtype == FEM_F64 && physics != FEM_ELASTICITY);
        e = launch_residual_lane(dim, physics, rule, coef_space, dtype, a, l);
    }
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_integrate_residual launch");
}

fem_status fem_integrate_residual_mesh(int dim, int physics, int rule, int coef_space, int dtype, int64_t n_elem,
                                       int64_t n_vert,
                                       const double* coords, const int32_t* conn, const void* u, const void* coef,
                                       void* elem_vec, void* inv_j, void* det_j, int32_t* counts, void* stream) {
    fem_status st = check_combo("fem_integrate_residual_mesh", dim, physics, rule, dtype);
    if (!st) st = check_space("fem_integrate_residual_mesh", coef_space);
    if (st) return st;
    if (n_elem < 0 || n_vert < 0) { set_error("fem_integrate_residual_mesh: negative size"); return FEM_ERR_INVALID_ARG; }
    if (n_elem == 0) return FEM_OK;
    if (n_vert == 0) { set_error("fem_integrate_residual_mesh: elements without vertices"); return FEM_ERR_INVALID_ARG; }
    if (!coords || !conn || !u || !coef || !elem_vec || (!inv_j) != (!det_j)) {
        set_error("fem_integrate_residual_mesh: NULL array (inv_j and det_j must both be set or both NULL)");
        return FEM_ERR_INVALID_ARG;
    }
    const fem_tuning t = get_tuning(FEM_OP_RESIDUAL_MESH, dim, physics, rule, dtype);
    MeshArgs a{n_elem, n_vert, coords, conn, u, coef, elem_vec, inv_j, det_j, counts};
    Launch l = make_tile_launch(t, n_elem, static_cast<hipStream_t>(stream));
    l.stream_out = whole_lines(n_elem, dtype == FEM_F32 ? 4 : 8, {elem_vec, inv_j, det_j});
    hipError_t e = t.strategy == FEM_STRATEGY_DEDUP ? launch_residual_dedup(dim, physics, rule, coef_space, dtype, a, l)
                                                    : launch_residual_mesh(dim, physics, rule, coef_space, dtype, a, l);
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_integrate_residual_mesh launch");
}

fem_status fem_integrate_residual_gather(int dim, int physics, int rule, int coef_space, int dtype, int64_t n_elem,
                                         int64_t n_vert, const double* coords, const int32_t* conn,
                                         const void* u_vertex, const void* coef, void* elem_vec, void* inv_j,
                                         void* det_j, int32_t* counts, void* stream) {
    fem_status st = check_combo("fem_integrate_residual_gather", dim, physics, rule, dtype);
    if (!st) st = check_space("fem_integrate_residual_gather", coef_space);
    if (st) return st;
    if (n_elem < 0 || n_vert < 0) { set_error("fem_integrate_residual_gather: negative size"); return FEM_ERR_INVALID_ARG; }
    if (n_elem == 0) return FEM_OK;
    if (n_vert == 0) { set_error("fem_integrate_residual_gather: elements without vertices"); return FEM_ERR_INVALID_ARG; }
    if (!coords || !conn || !u_vertex || !coef || !elem_vec || (!inv_j) != (!det_j)) {
        set_error("fem_integrate_residual_gather: NULL array (inv_j and det_j must both be set or both NULL)");
        return FEM_ERR_INVALID_ARG;
    }
    const fem_tuning t = get_tuning(FEM_OP_RESIDUAL_GATHER, dim, physics, rule, dtype);
    MeshArgs a{n_elem, n_vert, coords, conn, u_vertex, coef, elem_vec, inv_j, det_j, counts};
    Launch l = make_tile_launch(t, n_elem, static_cast<hipStream_t>(stream));
    // Three rows of a scalar form on triangles stream at odd words too, from 20 MiB on
    // (us streaming and plain: FP32, 1,000,003 triangles 11.9 and 11.2, 2,000,011 19.5
    // and 20.9, 3,000,017 28.6 and 29.7; FP64, 1,000,003 the same, 3,000,017 41.4 and
    // 44.0)
    const size_t word = dtype == FEM_F32 ? 4 : 8;
    const bool few = dim == 2 && physics != FEM_ELASTICITY && n_elem * (int64_t)word * 3 >= (int64_t)20 << 20;
    l.stream_out = few || whole_lines(n_elem, word, {elem_vec, inv_j, det_j});
    hipError_t e = launch_residual_gather(dim, physics, rule, coef_space, dtype, a, l);
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_integrate_residual_gather launch");
}

fem_status fem_integrate_residual_backward(int dim, int physics, int rule, int coef_space, int dtype, int64_t n_elem,
                                           const void* inv_j, const void* det_j, const void* u, const void* coef,
                                           const void* w, void* du, void* dcoef, void* stream) {
    fem_status st = check_combo("fem_integrate_residual_backward", dim, physics, rule, dtype);
    if (!st) st = check_space("fem_integrate_residual_backward", coef_space);
    if (st) return st;
    if (n_elem < 0) { set_error("fem_integrate_residual_backward: negative n_elem"); return FEM_ERR_INVALID_ARG; }
    if (n_elem == 0 || (!du && !dcoef)) return FEM_OK;
    if (!inv_j || !det_j || !w || (du && !coef) || (dcoef && !u)) {
        set_error("fem_integrate_residual_backward: NULL array");
        return FEM_ERR_INVALID_ARG;
    }
    bool chosen;
    fem_tuning t = get_tuning(FEM_OP_BACKWARD, dim, physics, rule, dtype, &chosen);
    const size_t word = dtype == FEM_F32 ? 4 : 8;
    const bool whole = whole_lines(n_elem, word, {du, dcoef});
    const int64_t pitch = n_elem * (int64_t)word;
    const int64_t rows = row_words(dim, physics, rule, coef_space, 1, (du ? 2 : 1) + (dcoef ? 1 : 0),
                                   (du ? 1 : 0) + (dcoef ? 1 : 0));
    if (!chosen) t = p1_tuning(t, dtype, n_elem, pitch * rows, whole,
                               whole_lines(n_elem, word, {inv_j, det_j, u, coef, w, du, dcoef}, 16));
    BackwardArgs a{n_elem, inv_j, det_j, u, coef, w, du, dcoef};
    Launch l = make_launch(t, (n_elem + t.vec - 1) / t.vec, t.vec, static_cast<hipStream_t>(stream));
    set_rows(l, whole, dim, dtype, pitch, rows, 1, true);
    hipError_t e = launch_backward_lane(dim, physics, rule, coef_space, dtype, a, l);
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_integrate_residual_backward launch");
}

fem_status fem_integrate_residual_p2(int dim, int physics, int rule, int coef_space, int dtype, int64_t n_elem,
                                     const void* inv_j, const void* det_j, const void* u, const void* coef,
                                     void* elem_vec, void* stream) {
    fem_status st = check_combo_p2("fem_integrate_residual_p2", dim, physics, rule, dtype);
    if (!st) st = check_space("fem_integrate_residual_p2", coef_space);
    if (st) return st;
    if (n_elem < 0) { set_error("fem_integrate_residual_p2: negative n_elem"); return FEM_ERR_INVALID_ARG; }
    if (n_elem == 0) return FEM_OK;
    if (!inv_j || !det_j || !u || !coef || !elem_vec) {
        set_error("fem_integrate_residual_p2: NULL array");
        return FEM_ERR_INVALID_ARG;
    }
    const fem_tuning t = get_tuning(FEM_OP_RESIDUAL_P2, dim, physics, rule, dtype);
    ResidualArgs a{n_elem, inv_j, det_j, u, coef, elem_vec};
    Launch l = make_launch(t, n_elem, 1, static_cast<hipStream_t>(stream));
    const size_t word = dtype == FEM_F32 ? 4 : 8;
    set_rows(l, whole_lines(n_elem, word, {elem_vec}), dim, dtype,
             n_elem * (int64_t)word, row_words(dim, physics, rule, coef_space, 2, 2, 1), 2, false);
    hipError_t e = launch_residual_p2(dim, physics, rule, coef_space, dtype, a, l);
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_integrate_residual_p2 launch");
}

fem_status fem_integrate_residual_p3(int dim, int physics, int rule, int coef_space, int dtype, int64_t n_elem,
                                     const void* inv_j, const void* det_j, const void* u, const void* coef,
                                     void* elem_vec, void* stream) {
    fem_status st = check_combo_p3("fem_integrate_residual_p3", dim, physics, rule, dtype);
    if (!st) st = check_space("fem_integrate_residual_p3", coef_space);
    if (st) return st;
    if (n_elem < 0) { set_error("fem_integrate_residual_p3: negative n_elem"); return FEM_ERR_INVALID_ARG; }
    if (n_elem == 0) return FEM_OK;
    if (!inv_j || !det_j || !u || !coef || !elem_vec) {
        set_error("fem_integrate_residual_p3: NULL array");
        return FEM_ERR_INVALID_ARG;
    }
    const fem_tuning t = get_tuning(FEM_OP_RESIDUAL_P3, dim, physics, rule, dtype);
    ResidualArgs a{n_elem, inv_j, det_j, u, coef, elem_vec};
    hipError_t e;
    if (t.strategy == FEM_STRATEGY_MFMA && mfma_available(FEM_OP_RESIDUAL_P3, dim, physics)) {
        // one wave per 16 elements
        Launch l = make_launch(t, (n_elem + 15) / 16 * 64, 1, static_cast<hipStream_t>(stream));
        e = launch_residual_p3_mfma(physics, coef_space, dtype, a, l);
    } else if (t.strategy == FEM_STRATEGY_COMPONENT && component_available(FEM_OP_RESIDUAL_P3, dim, physics)) {
        // three waves per 64-element tile; waves_per_block counts the
        // three-wave groups of a workgroup
        fem_tuning tg = t;
        tg.waves_per_block = 3 * t.waves_per_block;
        Launch l = make_launch(tg, (n_elem + 63) / 64 * 192, 1, static_cast<hipStream_t>(stream));
        e = launch_residual_p3_comp(coef_space, dtype, a, l);
    } else {
        Launch l = make_launch(t, n_elem, 1, static_cast<hipStream_t>(stream));
        const size_t word = dtype == FEM_F32 ? 4 : 8;
        set_rows(l, whole_lines(n_elem, word, {elem_vec}), dim, dtype,
                 n_elem * (int64_t)word, row_words(dim, physics, rule, coef_space, 3, 2, 1), 3, false,
                 physics == FEM_ELASTICITY && (dim == 3 || dtype == FEM_F64));
        e = launch_residual_p3(dim, physics, coef_space, dtype, a, l);
    }
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_integrate_residual_p3 launch");
}

fem_status fem_integrate_residual_p2_backward(int dim, int physics, int rule, int coef_space, int dtype,
                                              int64_t n_elem, const void* inv_j, const void* det_j, const void* u,
                                              const void* coef, const void* w, void* du, void* dcoef, void* stream) {
    fem_status st = check_combo_p2("fem_integrate_residual_p2_backward", dim, physics, rule, dtype);
    if (!st) st = check_space("fem_integrate_residual_p2_backward", coef_space);
    if (st) return st;
    if (n_elem < 0) { set_error("fem_integrate_residual_p2_backward: negative n_elem"); return FEM_ERR_INVALID_ARG; }
    if (n_elem == 0 || (!du && !dcoef)) return FEM_OK;
    if (!inv_j || !det_j || !w || (du && !coef) || (dcoef && !u)) {
        set_error("fem_integrate_residual_p2_backward: NULL array");
        return FEM_ERR_INVALID_ARG;
    }
    const fem_tuning t = get_tuning(FEM_OP_BACKWARD_P2, dim, physics, rule, dtype);
    BackwardArgs a{n_elem, inv_j, det_j, u, coef, w, du, dcoef};
    Launch l = make_launch(t, n_elem, 1, static_cast<hipStream_t>(stream));
    const size_t word = dtype == FEM_F32 ? 4 : 8;
    set_rows(l, whole_lines(n_elem, word, {du, dcoef}), dim, dtype,
             n_elem * (int64_t)word, row_words(dim, physics, rule, coef_space, 2, (du ? 2 : 1) + (dcoef ? 1 : 0), (du ? 1 : 0) + (dcoef ? 1 : 0)), 2, true);
    hipError_t e = launch_backward_p2(dim, physics, rule, coef_space, dtype, a, l);
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_integrate_residual_p2_backward launch");
}

fem_status fem_integrate_residual_p3_backward(int dim, int physics, int rule, int coef_space, int dtype,
                                              int64_t n_elem, const void* inv_j, const void* det_j, const void* u,
                                              const void* coef, const void* w, void* du, void* dcoef, void* stream) {
    fem_status st = check_combo_p3("fem_integrate_residual_p3_backward", dim, physics, rule, dtype);
    if (!st) st = check_space("fem_integrate_residual_p3_backward", coef_space);
    if (st) return st;
    if (n_elem < 0) { set_error("fem_integrate_residual_p3_backward: negative n_elem"); return FEM_ERR_INVALID_ARG; }
    if (n_elem == 0 || (!du && !dcoef)) return FEM_OK;
    if (!inv_j || !det_j || !w || (du && !coef) || (dcoef && !u)) {
        set_error("fem_integrate_residual_p3_backward: NULL array");
        return FEM_ERR_INVALID_ARG;
    }
    const fem_tuning t = get_tuning(FEM_OP_BACKWARD_P3, dim, physics, rule, dtype);
    BackwardArgs a{n_elem, inv_j, det_j, u, coef, w, du, dcoef};
    Launch l = make_launch(t, n_elem, 1, static_cast<hipStream_t>(stream));
    const size_t word = dtype == FEM_F32 ? 4 : 8;
    set_rows(l, whole_lines(n_elem, word, {du, dcoef}), dim, dtype,
             n_elem * (int64_t)word, row_words(dim, physics, rule, coef_space, 3, (du ? 2 : 1) + (dcoef ? 1 : 0), (du ? 1 : 0) + (dcoef ? 1 : 0)), 3, true);
    hipError_t e = launch_backward_p3(dim, physics, coef_space, dtype, a, l);
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_integrate_residual_p3_backward launch");
}

fem_status fem_integrate_jacobian(int dim, int physics, int rule, int coef_space, int order, int dtype,
                                  int64_t n_elem, const void* inv_j, const void* det_j, const void* coef,
                                  void* elem_mat, void* stream) {
    fem_status st = check_combo_jac("fem_integrate_jacobian", dim, physics, order, rule, dtype);
    if (!st) st = check_space("fem_integrate_jacobian", coef_space);
    if (st) return st;
    if (n_elem < 0) { set_error("fem_integrate_jacobian: negative n_elem"); return FEM_ERR_INVALID_ARG; }
    if (n_elem == 0) return FEM_OK;
    if (!inv_j || !det_j || !coef || !elem_mat) {
        set_error("fem_integrate_jacobian: NULL array");
        return FEM_ERR_INVALID_ARG;
    }
    const int op = order == 1 ? FEM_OP_JACOBIAN : order == 2 ? FEM_OP_JACOBIAN_P2 : FEM_OP_JACOBIAN_P3;
    bool chosen;
    fem_tuning t = get_tuning(op, dim, physics, rule, dtype, &chosen);
    // Rows at odd words: four waves per workgroup, XCD by XCD. Whole lines in
    // launch order (P1 3D elasticity FP64, one element per lane: 400,000 tets 113
    // us, 115 us XCD by XCD; 400,001 tets 184 us streaming in launch order, 145
    // us this way), but P1 elasticity rows of 4 MiB or more, whose kernels give a
    // lane 16 bytes of a row, four waves and XCD by XCD as well: 3D FP64, 327,680
    // tets 86 us, 88 this way, 524,288 tets 138 and 135, 2^21 tets 569 and 544; 2D
    // FP32, 2^21 triangles 81 and 77.
    const size_t word = dtype == FEM_F32 ? 4 : 8;
    const bool whole = whole_lines(n_elem, word, {elem_mat});
    const bool by_xcd = !whole || (order == 1 && physics == FEM_ELASTICITY && n_elem * (int64_t)word >= (int64_t)4 << 20);
    // P2 scalar rows a multiple of 8 MiB apart take four waves too, from 512 MiB on (3D Laplacian
    // FP64, 2^20 tets 200 us with one, 193 with four; 10^6 tets 190 either way).
    const int64_t pitch = n_elem * (int64_t)word, nb = (dim + 1) * (dim + 2) / 2;
    const bool apart = order == 2 && physics != FEM_ELASTICITY && pitch % ((int64_t)8 << 20) == 0 && pitch * nb * nb >= (int64_t)512 << 20;
    if ((by_xcd || apart) && !chosen) t = fem_tuning{FEM_STRATEGY_LANE, 1, 4, 0};
    JacobianArgs a{n_elem, inv_j, det_j, coef, elem_mat};
    Launch l = make_launch(t, n_elem, 1, static_cast<hipStream_t>(stream));
    l.stream_out = whole;
    l.order = by_xcd ? kOrderXcd : kOrderLaunch;
    hipError_t e = order == 3 ? launch_jacobian_p3(dim, physics, coef_space, dtype, a, l)
                              : launch_jacobian(dim, physics, order, rule, coef_space, dtype, a, l);
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_integrate_jacobian launch");
}

fem_status fem_stream_copy(const void* src, void* dst, int64_t n_bytes, void* stream) {
    if (n_bytes < 0 || (n_bytes % 16) || (reinterpret_cast<uintptr_t>(src) % 16) ||
        (reinterpret_cast<uintptr_t>(dst) % 16)) {
        set_error("fem_stream_copy: sizes and pointers must be multiples of 16 bytes");
        return FEM_ERR_INVALID_ARG;
    }
    if (n_bytes == 0) return FEM_OK;
    if (!src || !dst) { set_error("fem_stream_copy: NULL pointer"); return FEM_ERR_INVALID_ARG; }
    fem_tuning t{FEM_STRATEGY_LANE, 1, 4, 0};
    Launch l = make_launch(t, n_bytes / 16, 1, static_cast<hipStream_t>(stream));
    hipError_t e = launch_stream_copy(src, dst, n_bytes, l);
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_stream_copy launch");
}

fem_status fem_stream_rows(int dtype, int64_t n, int n_in, int n_out, const void* src, void* dst, void* stream) {
    if (!valid_dtype(dtype)) { set_error("fem_stream_rows: unknown dtype %d", dtype); return FEM_ERR_UNSUPPORTED; }
    if (n < 0 || n_in < 1 || n_in > FEM_STREAM_ROWS_MAX || n_out < 1 || n_out > FEM_STREAM_ROWS_MAX) {
        set_error("fem_stream_rows: n must be >= 0 and the row counts in 1..%d", FEM_STREAM_ROWS_MAX);
        return FEM_ERR_INVALID_ARG;
    }
    if (n == 0) return FEM_OK;
    if (!src || !dst) { set_error("fem_stream_rows: NULL pointer"); return FEM_ERR_INVALID_ARG; }
    fem_tuning t{FEM_STRATEGY_LANE, 1, 4, 0};
    Launch l = make_launch(t, n, 1, static_cast<hipStream_t>(stream));
    hipError_t e = launch_stream_rows(dtype, n, n_in, n_out, src, dst, l);
    return e == hipSuccess ? FEM_OK : hip_fail(e, "fem_stream_rows launch");
}

}  // extern "C"
