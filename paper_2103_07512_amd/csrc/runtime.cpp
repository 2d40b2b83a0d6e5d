// runtime.cpp -- host side of libtgp: contexts, domains, the population DAG,
// the cache planner, the program emitter and the C ABI of include/tgp.h.
//
// Evaluation of a DAG over a domain (TensorGP Sec. 3.1, with the subtree
// caching of Sec. 1 / Sec. 2) is planned on the host:
//   * every distinct (root, channel) pair becomes one interpreter program;
//   * a shared subtree is materialised once in an HBM cache row when
//     re-computing it at each use costs more VALU work than writing the row
//     once and reading it at each use (HBM traffic priced in VALU slots);
//   * on a grid with rows and columns, a subtree that depends on one of the
//     two alone is evaluated once per row or column into a table;
//   * subtrees whose evaluation would need more stack slots than the
//     interpreter keeps in registers are materialised as well, so every
//     program fits the register stack;
//   * cached subtrees are filled level by level (a row's program may read
//     rows of lower levels), then the root programs run fused with the error
//     reduction (fitness) or with a store of their values (evaluate).
#include <hip/hip_runtime.h>

#include <sched.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <array>
#include <atomic>
#include <chrono>
#include <cmath>
#include <functional>
#include <memory>
#include <mutex>
#include <string>
#include <system_error>
#include <thread>
#include <unordered_map>
#include <vector>

#include "runtime_internal.h"

namespace tgp {
extern uint32_t g_debug_hash_bits;
}

// ------------------------------------------------------------------ errors
static thread_local std::string g_err;

hipError_t ctx_pinned(tgp_ctx ctx, size_t bytes, void **out) {
    if (ctx->pin_pending) {
        hipError_t e = hipEventSynchronize(ctx->pin_ev);
        if (e != hipSuccess) return e;
        ctx->pin_pending = false;
    }
    if (ctx->pin_cap < bytes) {
        if (ctx->pin) hipHostFree(ctx->pin);
        ctx->pin = nullptr;
        ctx->pin_cap = 0;
        size_t want = 1 << 20;
        while (want < bytes) want <<= 1;
        hipError_t e = hipHostMalloc(&ctx->pin, want, hipHostMallocDefault);
        if (e != hipSuccess) return e;
        ctx->pin_cap = want;
    }
    *out = ctx->pin;
    return hipSuccess;
}

hipError_t ctx_pinned_enqueued(tgp_ctx ctx) {
    if (!ctx->pin_ev) {
        hipError_t e = hipEventCreateWithFlags(&ctx->pin_ev, hipEventDisableTiming);
        if (e != hipSuccess) return e;
    }
    hipError_t e = hipEventRecord(ctx->pin_ev, ctx->stream);
    if (e == hipSuccess) ctx->pin_pending = true;
    return e;
}

tgp_status fail(tgp_ctx ctx, tgp_status st, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (ctx) ctx->err = buf;
    g_err = buf;
    return st;
}

// The device code looks arities up in a packed constant; it must agree with
// the table for every opcode.
constexpr bool packed_arities_match() {
    for (int i = 0; i < TGP_NUM_OPS; ++i)
        if (arity_of((uint32_t)i) != kArityList[i] || kArityList[i] > 3) return false;
    return true;
}
static_assert(packed_arities_match(), "every arity fits two bits and unpacks to the table's value");

// --------------------------------------------------------------- cost model
// The planner's estimate of each operator's cost in VALU instructions per
// case, first measured with one-operator kernels over random inputs in
// [-1, 1] (SQ_INSTS_VALU less loads, stores and indexing) on earlier
// implementations of the operators; pow, mod, exp, log and sqrt have fast
// paths since and cost less, which only makes the planner cache a little
// more of them than it would.  Terminals cost the register move that places
// them on the stack; warp is estimated (two axis points and a gathered
// read).  It steers caching and program order only; reported throughput
// does not use it.
const double kOpCost[TGP_NUM_OPS] = {
    1,  1,              // var const
    1,  1,  1, 13,      // add sub mult div
    38, 35, 55,         // sin cos tan
    14, 15, 83,         // exp log pow
    3,  3,  3,  1,      // min max mdist neg
    19, 4,  1,  5,      // sqrt sign abs clip
    42, 2,  2,          // mod frac if
    2,  6,  9, 27, 9,   // step sstep sstepp len lerp
    16, 16, 16,         // or xor and
    24                  // warp
};
// Writing a cache row once and reading it back, in VALU-slot equivalents per
// case: 4 bytes of HBM traffic at 8 TB/s against 256 CUs x 64 lanes x 2.4 GHz
// of VALU issue is about 20 slots per access (the default of
// tgp_ctx_set_plan's cache_access_cost).

// ------------------------------------------------- fixed device scratch
// tgp_fitness_noalloc keeps its partial sums and subtree cache rows in this
// array instead of allocated buffers, so it calls no allocator.  Each GPU
// the library runs on holds its own copy until the process ends.  In host
// code `scratch` only names the symbol: its device address is looked up once
// per device (hipGetSymbolAddress, at context creation, with the device
// current) and that address is what kernels and copies receive.
constexpr size_t kNoAllocScratchBytes = size_t(64) << 20;
// Smallest domain evaluated by table programs (a smaller one is a few waves
// per program either way, and the tables cost a launch).
constexpr int64_t kTableCases = 1024;
// A DAG below so many nodes has few cached rows, if any, so its tables are a
// launch more, which pays from so many node-evals on.  A planned call, flat and
// with tables, us (alone; one of many): 4 nodes on 512^2 cases 19.5 and 21.2 (8.6
// and 11.8), 34 nodes 20.6 and 22.5 (9.3 and 13.5), 79 nodes 24.0 and 24.7 (12.3
// and 14.9); on 1024^2 34 nodes 30.6 and 31.1, 47 nodes 33.5 and 31.9, 79 nodes
// 43.4 and 39.9; 118 nodes on 64^2 27.4 and 24.6 (15.9 and 15.7).
constexpr int64_t kTableNodes = 100, kTableWork = int64_t(1) << 25;
__device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices];
hipError_t g_scratch_err[kMaxDevices];
}  // namespace

// With `device` current: its scratch address, looked up on first use.
static void scratch_setup(int device) {
    if (device < 0 || device >= kMaxDevices) return;
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (g_scratch_ptr[device]) return;
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    g_scratch_err[device] = e;
    if (e == hipSuccess) g_scratch_ptr[device] = p;
    else (void)hipGetLastError();  // leave no error behind for the next call
}

// --------------------------------------------------------------- contexts
extern "C" {

tgp_status tgp_ctx_create(int device, void *hip_stream, tgp_ctx *out) {
    if (!out) return fail(nullptr, TGP_EINVAL, "out is NULL");
    *out = nullptr;
    int n = 0;
    hipError_t e = hipGetDeviceCount(&n);
    if (e != hipSuccess || n == 0)
        return fail(nullptr, TGP_EHIP, "no HIP device: %s", hipGetErrorString(e));
    if (device < 0 || device >= n) return fail(nullptr, TGP_EINVAL, "device %d out of range", device);
    e = hipSetDevice(device);
    if (e != hipSuccess) return fail(nullptr, TGP_EHIP, "hipSetDevice: %s", hipGetErrorString(e));
    hipDeviceProp_t prop;
    e = hipGetDeviceProperties(&prop, device);
    if (e != hipSuccess)
        return fail(nullptr, TGP_EHIP, "hipGetDeviceProperties: %s", hipGetErrorString(e));
    if (strncmp(prop.gcnArchName, "gfx950", 6) != 0)
        return fail(nullptr, TGP_EHIP, "device %d is %s, libtgp is built for gfx950", device,
                    prop.gcnArchName);
    scratch_setup(device);
    tgp_ctx c = new tgp_ctx_s();
    c->device = device;
    c->stream = (hipStream_t)hip_stream;
    c->cache_budget = prop.totalGlobalMem / 4;
    *out = c;
    return TGP_OK;
}

void tgp_ctx_destroy(tgp_ctx ctx) {
    if (!ctx) return;
    hipSetDevice(ctx->device);
    hipStreamSynchronize(ctx->stream);
    tgp_batch_destroy(ctx->batch);
    hipFree(ctx->partial.p);
    hipFree(ctx->cache.p);
    hipFree(ctx->tables.p);
    hipFree(ctx->fit_out.p);
    ctx->pool.drain();
    if (ctx->pin) hipHostFree(ctx->pin);
    if (ctx->pin_ev) hipEventDestroy(ctx->pin_ev);
    if (ctx->ev_ready)
        for (auto &e : ctx->ev) hipEventDestroy(e);
    delete ctx;
}

tgp_status tgp_ctx_set_stream(tgp_ctx ctx, void *hip_stream) {
    if (!ctx) return fail(nullptr, TGP_EINVAL, "ctx is NULL");
    ctx->stream = (hipStream_t)hip_stream;
    return TGP_OK;
}

const char *tgp_last_error(tgp_ctx ctx) { return ctx ? ctx->err.c_str() : g_err.c_str(); }

tgp_status tgp_ctx_set_cache_budget(tgp_ctx ctx, size_t bytes) {
    if (!ctx) return fail(nullptr, TGP_EINVAL, "ctx is NULL");
    ctx->cache_budget = bytes;
    return TGP_OK;
}

tgp_status tgp_ctx_set_timing(tgp_ctx ctx, int32_t enable) {
    if (!ctx) return fail(nullptr, TGP_EINVAL, "ctx is NULL");
    if (enable && !ctx->ev_ready) {
        HCHK(ctx, hipSetDevice(ctx->device));
        for (auto &e : ctx->ev) HCHK(ctx, hipEventCreate(&e));
        ctx->ev_ready = true;
    }
    ctx->timing = enable != 0;
    return TGP_OK;
}

tgp_status tgp_last_timing(tgp_ctx ctx, tgp_timing *out) {
    if (!ctx || !out) return fail(ctx, TGP_EINVAL, "NULL argument");
    tgp_timing t = ctx->times;
    t.fill_ms = t.interp_ms = t.finalize_ms = 0;
    t.breed_shape_ms = t.breed_plan_ms = t.breed_write_ms = 0;
    if (ctx->timing && ctx->ev_ready) {
        // device time between two recorded events (0 when one never was)
        auto span = [ctx](int a, int b, double *out) -> hipError_t {
            if (!(ctx->recorded >> a & 1u) || !(ctx->recorded >> b & 1u)) return hipSuccess;
            hipError_t e = hipEventSynchronize(ctx->ev[b]);
            float ms = 0;
            if (e == hipSuccess) e = hipEventElapsedTime(&ms, ctx->ev[a], ctx->ev[b]);
            if (e == hipSuccess) *out = ms;
            return e;
        };
        if (ctx->fill_recorded) HCHK(ctx, span(0, 1, &t.fill_ms));
        HCHK(ctx, span(2, 3, &t.interp_ms));
        HCHK(ctx, span(4, 5, &t.finalize_ms));
        HCHK(ctx, span(6, 7, &t.breed_shape_ms));
        HCHK(ctx, span(7, 8, &t.breed_plan_ms));
        HCHK(ctx, span(9, 10, &t.breed_write_ms));
    }
    *out = t;
    return TGP_OK;
}

// Tuning knobs (used by the autotuner and tests): cases per lane (2 or 4, 0 =
// automatic) and tiles per work item (0 = automatic).
tgp_status tgp_ctx_set_tuning(tgp_ctx ctx, int32_t cases_per_lane, int32_t tiles_per_item) {
    if (!ctx) return fail(nullptr, TGP_EINVAL, "ctx is NULL");
    if (cases_per_lane != 0 && !interp_variant_exists(cases_per_lane, interp_max_stack()))
        return fail(ctx, TGP_EINVAL, "no interpreter with %d cases per lane", cases_per_lane);
    if (tiles_per_item < 0) return fail(ctx, TGP_EINVAL, "tiles_per_item < 0");
    ctx->force_K = cases_per_lane;
    ctx->force_tiles = tiles_per_item;
    ctx->tile_cap = 0;
    return TGP_OK;
}

tgp_status tgp_ctx_set_hashing(tgp_ctx ctx, int32_t commutative) {
    if (!ctx) return fail(nullptr, TGP_EINVAL, "ctx is NULL");
    ctx->commute = commutative != 0;
    return TGP_OK;
}

tgp_status tgp_ctx_set_rewrite(tgp_ctx ctx, int32_t on) {
    if (!ctx) return fail(nullptr, TGP_EINVAL, "ctx is NULL");
    ctx->rewrite = on != 0;
    return TGP_OK;
}

tgp_status tgp_ctx_set_folding(tgp_ctx ctx, int32_t on) {
    if (!ctx) return fail(nullptr, TGP_EINVAL, "ctx is NULL");
    ctx->fold = on != 0;
    return TGP_OK;
}

tgp_status tgp_ctx_set_stack(tgp_ctx ctx, int32_t lds) {
    if (!ctx) return fail(nullptr, TGP_EINVAL, "ctx is NULL");
    ctx->stack_lds = lds != 0;
    return TGP_OK;
}

tgp_status tgp_ctx_set_plan(tgp_ctx ctx, int32_t reorder_children, double cache_access_cost) {
    if (!ctx) return fail(nullptr, TGP_EINVAL, "ctx is NULL");
    ctx->reorder = reorder_children != 0;
    ctx->cache_access_cost = cache_access_cost;
    return TGP_OK;
}

tgp_status tgp_debug_set_hash_bits(int32_t bits) {
    if (bits < 0 || bits > 32) return fail(nullptr, TGP_EINVAL, "bits must be 0..32");
    g_debug_hash_bits = (uint32_t)bits;
    return TGP_OK;
}

// ---------------------------------------------------------------- domains
}  // extern "C"

// Where table programs split the axes of a domain (0: nowhere, it is
// evaluated flat).  Either side must hold at least 8 entries, so that a table
// entry costs at most an eighth of evaluating its subtree at every case, and
// the domain at least kTableCases cases.  Columns in multiples of kWideCols
// make the wide form; otherwise the split with the shorter tables is taken.
static int32_t domain_split(const tgp_domain_s &d) {
    if (d.cases < kTableCases) return 0;
    int best = 0;
    double best_score = 0;
    for (int s = d.ndim - 1; s >= 1; --s) {
        const int64_t r = d.rows(s), c = d.cols(s);
        if (r < 8 || c < 8) continue;
        const double score = 1.0 / (double)(r + c) + (c % kWideCols == 0 ? 1.0 : 0.0);
        if (score > best_score) {
            best = s;
            best_score = score;
        }
    }
    return best;
}

extern "C" {
tgp_status tgp_domain_create(tgp_ctx ctx, int32_t ndim, const int64_t *shape, const double *lo,
                             const double *hi, tgp_domain *out) {
    if (!ctx || !out || !shape) return fail(ctx, TGP_EINVAL, "NULL argument");
    *out = nullptr;
    if (ndim < 1 || ndim > 3) return fail(ctx, TGP_ESHAPE, "ndim must be 1..3, got %d", ndim);
    int64_t cases = 1;
    for (int k = 0; k < ndim; ++k) {
        if (shape[k] < 1) return fail(ctx, TGP_ESHAPE, "shape[%d] = %lld < 1", k, (long long)shape[k]);
        cases *= shape[k];
        if (cases > (1LL << 30)) return fail(ctx, TGP_ESHAPE, "more than 2^30 cases");
    }
    HCHK(ctx, hipSetDevice(ctx->device));
    tgp_domain d = new tgp_domain_s();
    d->ctx = ctx;
    d->ndim = ndim;
    d->cases = cases;
    int64_t st = 1;
    for (int k = ndim - 1; k >= 0; --k) {
        d->shape[k] = shape[k];
        d->stride[k] = st;
        st *= shape[k];
    }
    for (int k = 0; k < ndim; ++k) {
        const double l = lo ? lo[k] : -1.0, h = hi ? hi[k] : 1.0;
        d->lo[k] = l;
        d->hi[k] = h;
        std::vector<float> tab(shape[k]);
        for (int64_t i = 0; i < shape[k]; ++i) {
            const double v = shape[k] == 1 ? l : l + (h - l) * (double)i / (double)(shape[k] - 1);
            tab[i] = (float)v;
        }
        hipError_t e = hipMalloc((void **)&d->coord[k], sizeof(float) * shape[k]);
        if (e == hipSuccess)
            e = hipMemcpy(d->coord[k], tab.data(), sizeof(float) * shape[k], hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            tgp_domain_destroy(d);
            return fail(ctx, TGP_EHIP, "coordinate table: %s", hipGetErrorString(e));
        }
    }
    d->split = domain_split(*d);
    *out = d;
    return TGP_OK;
}

void tgp_domain_destroy(tgp_domain d) {
    if (!d) return;
    for (int k = 0; k < 3; ++k) hipFree(d->coord[k]);
    delete d;
}

int64_t tgp_domain_cases(tgp_domain d) { return d ? d->cases : -1; }

// -------------------------------------------------------------------- DAG
tgp_status tgp_build_dag(tgp_ctx ctx, const tgp_population *pop, tgp_dag *out) {
    if (!ctx || !pop || !out) return fail(ctx, TGP_EINVAL, "NULL argument");
    *out = nullptr;
    const double t0 = now_ms();
    if (pop->n_individuals < 0 || pop->n_channels < 1)
        return fail(ctx, TGP_EINVAL, "n_individuals < 0 or n_channels < 1");
    if (pop->memory != TGP_MEM_HOST && pop->memory != TGP_MEM_DEVICE)
        return fail(ctx, TGP_EINVAL, "memory must be TGP_MEM_HOST or TGP_MEM_DEVICE");
    const int64_t R = (int64_t)pop->n_individuals * pop->n_channels;
    if (R > 0 && (!pop->offsets || !pop->tokens)) return fail(ctx, TGP_EINVAL, "NULL offsets/tokens");
    HCHK(ctx, hipSetDevice(ctx->device));
    int64_t T = 0;
    const int64_t *off_dev = nullptr;
    const tgp_token *tok_dev = nullptr;
    int64_t *off_own = nullptr;
    tgp_token *tok_own = nullptr;
    if (R > 0) {
        if (pop->memory == TGP_MEM_HOST) {
            if (pop->offsets[0] != 0) return fail(ctx, TGP_EINVAL, "offsets[0] must be 0");
            for (int64_t r = 0; r < R; ++r)
                if (pop->offsets[r + 1] < pop->offsets[r])
                    return fail(ctx, TGP_EINVAL, "offsets decrease at tree %lld", (long long)r);
            T = pop->offsets[R];
            if (T > 0x7fffffffLL) return fail(ctx, TGP_EINVAL, "more than 2^31-1 tokens");
            // offsets and tokens in one block, through the pinned staging
            const size_t ob = sizeof(int64_t) * (R + 1), tb = sizeof(tgp_token) * T;
            void *stage = nullptr;
            HCHK(ctx, ctx->pool.alloc((void **)&off_own, ob + tb));
            tok_own = reinterpret_cast<tgp_token *>(off_own + R + 1);
            HCHK(ctx, ctx_pinned(ctx, ob + tb, &stage));
            memcpy(stage, pop->offsets, ob);
            if (T) memcpy((char *)stage + ob, pop->tokens, tb);
            HCHK(ctx, hipMemcpyAsync(off_own, stage, ob + tb, hipMemcpyHostToDevice, ctx->stream));
            HCHK(ctx, ctx_pinned_enqueued(ctx));
            off_dev = off_own;
            tok_dev = tok_own;
        } else {
            T = -1;  // read from offsets[R] by the build
            off_dev = pop->offsets;
            tok_dev = pop->tokens;
        }
    }
    tgp_dag d = new tgp_dag_s();
    d->ctx = ctx;
    d->n_ind = pop->n_individuals;
    d->n_ch = pop->n_channels;
    d->stats.n_roots = R;
    d->stats.max_var = -1;
    if (R > 0) {
        char msg[256] = "";
        const int32_t *h = nullptr;
        DagBuildResult br = build_dag_device(ctx, tok_dev, off_dev, R, T, &d->dev, &h, msg, sizeof msg);
        ctx->pool.release(off_own);  // build_dag_device has synchronised the stream
        if (br.status != TGP_OK) {
            delete d;
            return fail(ctx, (tgp_status)br.status, "build_dag: %s", msg);
        }
        const int64_t U = br.U;
        d->swap(ctx->spare_dag);
        d->op.resize(U);
        d->value.resize(U);
        d->kid.resize(3 * U);
        d->height.resize(U);
        d->roots.resize(R);
        d->mult.resize(U);
        d->indeg.resize(U);
        memcpy(d->op.data(), h, sizeof(int32_t) * U);
        memcpy(d->value.data(), h + U, sizeof(float) * U);
        memcpy(d->kid.data(), h + 2 * U, sizeof(int32_t) * 3 * U);
        memcpy(d->height.data(), h + 5 * U, sizeof(int32_t) * U);
        memcpy(d->mult.data(), h + 6 * U, sizeof(int32_t) * U);
        memcpy(d->indeg.data(), h + 7 * U, sizeof(int32_t) * U);
        memcpy(d->roots.data(), h + 8 * U, sizeof(int32_t) * R);
        d->stats.tree_nodes = br.T;
        d->stats.tree_internal = br.tree_internal;
        d->stats.dag_nodes = U;
        int64_t di = 0, sh = 0;
        for (int64_t i = 0; i < U; ++i) {
            const int op = d->op[i] & 0xff;
            if (kArity[op] > 0) {
                ++di;
                if (d->mult[i] >= 2) ++sh;
            }
            d->image_ops |= op == TGP_WARP || op == TGP_OR || op == TGP_XOR || op == TGP_AND;
        }
        d->stats.dag_internal = di;
        d->stats.shared_internal = sh;
        d->stats.max_stack = br.max_stack;
        d->stats.max_height = br.max_height;
        d->stats.max_var = br.max_var;
    }
    *out = d;
    ctx->times.build_dag_ms = now_ms() - t0;
    return TGP_OK;
}

tgp_status tgp_dag_stats_get(tgp_dag dag, tgp_dag_stats *out) {
    if (!dag || !out) return fail(nullptr, TGP_EINVAL, "NULL argument");
    *out = dag->stats;
    return TGP_OK;
}

tgp_status tgp_dag_export(tgp_dag dag, tgp_token *nodes, int32_t *children, int32_t *roots,
                          int32_t *multiplicity, int32_t *indegree) {
    if (!dag) return fail(nullptr, TGP_EINVAL, "dag is NULL");
    const int64_t U = dag->stats.dag_nodes;
    if (nodes)
        for (int64_t i = 0; i < U; ++i) {
            nodes[i].op = (uint8_t)(dag->op[i] & 0xff);
            nodes[i].var = (uint8_t)((dag->op[i] >> 8) & 0xff);
            nodes[i].pad = 0;
            nodes[i].value = dag->value[i];
        }
    if (children && U) memcpy(children, dag->kid.data(), sizeof(int32_t) * 3 * U);
    if (roots && dag->stats.n_roots) memcpy(roots, dag->roots.data(), sizeof(int32_t) * dag->stats.n_roots);
    if (multiplicity && U) memcpy(multiplicity, dag->mult.data(), sizeof(int32_t) * U);
    if (indegree && U) memcpy(indegree, dag->indeg.data(), sizeof(int32_t) * U);
    return TGP_OK;
}

void tgp_dag_destroy(tgp_dag dag) {
    if (!dag) return;
    tgp_ctx ctx = dag->ctx;
    hipSetDevice(ctx->device);
    hipStreamSynchronize(ctx->stream);  // no queued kernel reads the blocks any more
    dag->plan.release(ctx->pool);
    dag->other.release(ctx->pool);
    dag_device_free(&dag->dev, ctx->pool);
    if (dag->op.capacity() > ctx->spare_dag.op.capacity()) dag->swap(ctx->spare_dag);
    for (Plan *P : {&dag->plan, &dag->other})
        if (P->code_host.capacity() > ctx->spare_code.capacity()) P->code_host.swap(ctx->spare_code);
    delete dag;
}

}  // extern "C"

// ------------------------------------------------------------------ planner
namespace {

// A spin-wait hint to the host processor.
inline void cpu_relax() {
#if defined(__x86_64__) || defined(__i386__)
    __builtin_ia32_pause();
#endif
}

}  // namespace

HostTeam::~HostTeam() {
    {
        std::lock_guard<std::mutex> lk(m_);
        stop_ = true;
    }
    cv_.notify_all();
    for (auto &t : workers_) t.join();
}

int HostTeam::grow(int T) {
    T = std::min(T, kMaxWorkers + 1);
    try {
        while ((int)workers_.size() < T - 1) {
            const int id = (int)workers_.size() + 1;
            workers_.emplace_back(&HostTeam::work, this, id, round_.load());
        }
    } catch (const std::system_error &) {  // no more threads to be had
    }
    return std::min(T, (int)workers_.size() + 1);
}

void HostTeam::run(int T, const std::function<void(int)> &fn) {
    {
        std::lock_guard<std::mutex> lk(m_);
        fn_ = &fn;
        want_ = T;
        left_.store(T - 1, std::memory_order_relaxed);
        round_.fetch_add(1, std::memory_order_release);
    }
    cv_.notify_all();
    fn(0);
    for (int i = 0; left_.load(std::memory_order_acquire) > 0; ++i) {
        if (i < 4000) cpu_relax();
        else std::this_thread::yield();
    }
}

// Worker id waits for a round it takes part in (spinning for some
// microseconds first: the phases of one plan follow each other closely).
void HostTeam::work(int id, uint64_t seen) {
    for (;;) {
        for (int i = 0; i < 2000 && round_.load(std::memory_order_acquire) == seen; ++i) cpu_relax();
        const std::function<void(int)> *fn = nullptr;
        {
            std::unique_lock<std::mutex> lk(m_);
            cv_.wait(lk, [&] { return stop_ || round_.load(std::memory_order_relaxed) != seen; });
            if (stop_) return;
            seen = round_.load(std::memory_order_relaxed);
            if (id < want_) fn = fn_;
        }
        if (!fn) continue;
        (*fn)(id);
        left_.fetch_sub(1, std::memory_order_release);
    }
}

namespace {

// Processors this process may use: its affinity mask (the machine's count
// when the mask cannot be read), capped by a CPU quota of its control group
// (cgroup v2 cpu.max, "quota period"), rounded up.  The planner's threads
// wait for each other level by level, so more threads than processors would
// only slow it down.
unsigned usable_cpus() {
    static const unsigned n = [] {
        unsigned c = std::max(1u, std::thread::hardware_concurrency());
        cpu_set_t set;
        if (sched_getaffinity(0, sizeof set, &set) == 0) c = (unsigned)std::max(1, CPU_COUNT(&set));
        if (FILE *f = fopen("/sys/fs/cgroup/cpu.max", "r")) {
            char quota[32] = "";
            long long period = 0;
            if (fscanf(f, "%31s %lld", quota, &period) == 2 && strcmp(quota, "max") != 0 && period > 0) {
                const long long q = atoll(quota);
                if (q > 0) c = std::min<unsigned>(c, (unsigned)std::max(1LL, (q + period - 1) / period));
            }
            fclose(f);
        }
        return c;
    }();
    return n;
}

// T, or how many threads the team can run when that is fewer.
int team_size(HostTeam *team, int T) { return team && T > 1 ? team->grow(T) : T; }

// Runs fn(t) for t = 0 .. T-1 (T from team_size) on the team's threads, or
// (without a team) on threads of its own; the caller's thread is t = 0.
template <class F>
void run_threads(HostTeam *team, int T, F &&fn) {
    if (T <= 1) {
        fn(0);
    } else if (team) {
        team->run(T, fn);
    } else {
        std::vector<std::thread> th;
        for (int t = 1; t < T; ++t) th.emplace_back([&, t] { fn(t); });
        fn(0);
        for (auto &x : th) x.join();
    }
}

// Runs fn(t, barrier) on T host threads as run_threads does;
// barrier() returns once all T threads have reached it.  A waiting thread
// spins for a few microseconds first (the threads of one level usually
// arrive close together), then yields its processor.
template <class F>
void run_team(HostTeam *team, int T, F &&fn) {
    std::atomic<int> arrived{0}, generation{0};
    auto barrier = [&]() {
        const int g = generation.load(std::memory_order_acquire);
        if (arrived.fetch_add(1, std::memory_order_acq_rel) + 1 == T) {
            arrived.store(0, std::memory_order_relaxed);
            generation.fetch_add(1, std::memory_order_acq_rel);
        } else {
            for (int i = 0; i < 2000 && generation.load(std::memory_order_acquire) == g; ++i)
                cpu_relax();
            while (generation.load(std::memory_order_acquire) == g) std::this_thread::yield();
        }
    };
    run_threads(team, T, [&](int t) { fn(t, barrier); });
}

// The nodes 0..U-1 ordered by height (id order within a height) on T
// threads: order[first[h] .. first[h+1]) are the nodes of height h.
void height_order(HostTeam *team, const int32_t *hgt, int64_t U, int T, std::vector<int32_t> &order,
                  std::vector<int64_t> &first) {
    std::vector<std::vector<int64_t>> hist(T);
    int32_t H = 0;
    order.resize(U);
    run_team(team, T, [&](int t, auto &barrier) {
        const int64_t b = U * t / T, e = U * (t + 1) / T;
        std::vector<int64_t> &c = hist[t];
        for (int64_t n = b; n < e; ++n) {
            if ((size_t)hgt[n] >= c.size()) c.resize(hgt[n] + 1, 0);
            ++c[hgt[n]];
        }
        barrier();
        if (t == 0) {
            for (int i = 0; i < T; ++i) H = std::max(H, (int32_t)hist[i].size() - 1);
            first.assign(H + 2, 0);
            int64_t at = 0;
            for (int32_t h = 0; h <= H; ++h) {
                first[h] = at;
                for (int i = 0; i < T; ++i) {
                    const int64_t k = (size_t)h < hist[i].size() ? hist[i][h] : 0;
                    if ((size_t)h < hist[i].size()) hist[i][h] = at;
                    at += k;
                }
            }
            first[H + 1] = at;
        }
        barrier();
        for (int64_t n = b; n < e; ++n) order[c[hgt[n]]++] = (int32_t)n;
    });
}

// Whether tables of so many entries, each of slots_per cache slots of
// slot_bytes, may be used: at most half the cache budget, and a 32-bit byte
// offset into either.  *slots: their size.
bool tables_fit(const int64_t (&entries)[2], const double (&slots_per)[2], double slot_bytes, size_t budget_slots,
                size_t *slots) {
    *slots = (size_t)std::ceil(entries[0] * slots_per[0] + entries[1] * slots_per[1]);
    if (*slots > budget_slots / 2) return false;
    for (int q = 0; q < 2; ++q)
        if (entries[q] * slots_per[q] * slot_bytes >= 0xffffff00u) return false;
    return true;
}

struct Planner {
    const tgp_dag_s &d;
    int D;
    size_t budget_slots;
    std::vector<uint8_t> cached;
    std::vector<uint8_t> pre;   // cached and already resident: read, never filled
    std::vector<uint8_t> perm;  // evaluation order of each node's children (index in kPerms)
    std::vector<int32_t> slot, level;
    std::vector<double> cost;
    int64_t spills = 0;

    bool reorder = true;
    double access_cost = 20.0;
    HostTeam *team = nullptr;  // the planning context's threads (null: own ones)

    // Table programs: programs of subtrees that depend on axes on both sides of the
    // split read every other variable-dependent subtree from a table, where it
    // is evaluated once per grid row or column instead of once per case (with
    // the same operators, so bit for bit the same value).  cls: bit 0, the
    // subtree depends on an axis below the split (grid rows), bit 1, on
    // another one (columns); a cached node of class 1 or 2 is a table entry.
    // A table entry's own program is self-contained, except that it reads the
    // nested entries (those that bound its stack) from lower levels.
    int split = 0;
    double table_slots_per[2] = {0, 0};  // a table entry's size in cache slots
    std::vector<uint8_t> cls, nested;
    size_t table_slots = 0;              // the tables' size in cache slots
    bool tables_over = false;            // the tables do not fit the budget

    Planner(const tgp_dag_s &dag, int stack, size_t slots) : d(dag), D(stack), budget_slots(slots) {}

    bool in_table(int64_t n) const { return split > 0 && (cls[n] == 1 || cls[n] == 2); }
    int axis(int64_t n) const { return (d.op[n] >> 8) & 0xff; }
    // the tables' size once every entry is marked; false: they do not fit
    bool set_table_slots(const int64_t (&entries)[2]) {
        for (int q = 0; q < 2; ++q) table_entries[q] = entries[q];
        tables_over = !tables_fit(entries, table_slots_per, slot_bytes, budget_slots, &table_slots);
        return !tables_over;
    }
    double slot_bytes = 0;               // bytes of a cache slot
    int64_t table_entries[2] = {0, 0};

    // nodes by height (filled by the parallel preparation or decisions)
    std::vector<int32_t> lorder;
    std::vector<int64_t> lfirst;
    std::vector<uint8_t> folded;  // constant subtrees replaced by their value
    std::vector<float> fold_val;
    // A node as the planner sees it (a folded node is a constant leaf).  An
    // absent child is node U, which costs nothing and needs no stack, so that
    // the passes below have few branches (random trees make them
    // unpredictable).
    struct Node {
        int32_t k[3];
        uint8_t op, ar;
    };
    std::vector<Node> node;
    // Stack slots a node needs as the child of a program that reads cached
    // values (g) or, in a table entry's own program, nested ones (t), and
    // whether that program's operators can fuse it.
    struct Need {
        uint8_t g, t, fuse_g, fuse_t;
    };
    std::vector<Need> need;
    std::vector<std::vector<uint2>> emitted;  // each emitting thread's programs
    std::vector<int64_t> uses;
    std::vector<int32_t> dep;
    double valu_dag = 0;  // cost-model slots of every DAG node once (unfolded)
    int op(int64_t n) const { return node[n].op; }
    int arity(int64_t n) const { return node[n].ar; }

    // Exchanges the arrays that a context keeps between plans.
    void swap_scratch(PlanScratch &o);

    void resize(int64_t U) {
        node.resize(U + 1);
        node[U] = Node{{(int32_t)U, (int32_t)U, (int32_t)U}, TGP_CONST, 0};
        cached.assign(U + 1, 0);
        pre.assign(U + 1, 0);
        cost.resize(U + 1);
        cost[U] = 0.0;
        perm.assign(U + 1, 0);
        need.resize(U + 1);
        need[U] = Need{0, 0, 0, 0};
        uses.assign(U + 1, 0);
        dep.assign(U + 1, 0);
        level.assign(U + 1, -1);
        slot.assign(U + 1, -1);
        cls.assign(split > 0 ? U + 1 : 0, 0);
        nested.assign(split > 0 ? U + 1 : 0, 0);
    }
    // The decisions of planned nodes end at node U - 1.
    void trim(int64_t U) {
        cached.resize(U);
        level.resize(U);
        slot.resize(U);
    }

    // Node n's record; returns its unfolded cost.
    double load(int64_t n, int64_t U) {
        const int o = d.op[n] & 0xff;
        const bool leaf = !folded.empty() && folded[n];
        Node &x = node[n];
        for (int j = 0; j < 3; ++j) {
            const int32_t c = d.kid[3 * n + j];
            x.k[j] = leaf || c < 0 ? (int32_t)U : c;
        }
        x.op = (uint8_t)(leaf ? TGP_CONST : o);
        x.ar = (uint8_t)(leaf ? 0 : kArity[o]);
        return kOpCost[o];
    }
    // Marks are made by several threads at once in the level-parallel passes.
    static bool mark(std::vector<uint8_t> &v, int64_t n) {  // returns whether n was not marked before
        if (__atomic_load_n(&v[n], __ATOMIC_RELAXED)) return false;
        return __atomic_exchange_n(&v[n], (uint8_t)1, __ATOMIC_RELAXED) == 0;
    }

    // Class and cost of node n from its children's, whether it stays resident
    // (its values over this domain are kept from an earlier evaluation and
    // recomputing them costs more than the read), and the table entries that
    // it reads when the plan has tables.
    void up_cost(int64_t n, bool resident, bool is_root) {
        const Node &x = node[n];
        double c = kOpCost[x.op];
        if (split > 0) {
            const uint8_t own = x.op == TGP_VAR ? (axis(n) < split ? 1 : 2) : 0;
            const uint8_t k0 = cls[x.k[0]], k1 = cls[x.k[1]], k2 = cls[x.k[2]];
            const uint8_t m = own | k0 | k1 | k2;
            cls[n] = m;
            if (m == 3) {
                for (int j = 0; j < 3; ++j) {
                    const bool tab = in_table(x.k[j]);
                    c += tab ? 1.0 : cost[x.k[j]];
                    if (tab) __atomic_store_n(&cached[x.k[j]], (uint8_t)1, __ATOMIC_RELAXED);
                }
            } else {
                c += cost[x.k[0]] + cost[x.k[1]] + cost[x.k[2]];
                if (m && is_root) __atomic_store_n(&cached[n], (uint8_t)1, __ATOMIC_RELAXED);
            }
        } else {
            c += cost[x.k[0]] + cost[x.k[1]] + cost[x.k[2]];
        }
        cost[n] = c;
        if (resident && d.precached[n] && x.ar > 0 && !in_table(n) && c > access_cost) cached[n] = pre[n] = 1;
    }

    // Stack need and child order of node n.  Children are evaluated in
    // decreasing order of the stack they need (Sethi-Ullman, a fused last
    // operand taking no slot: x, y, a constant or a value read from a row
    // under an operator with a fused form); a node whose children still
    // cannot be evaluated within D slots gets its most demanding child's
    // subtree spilled: spill(child) is called, once per spilled child.
    template <class S>
    void up_need(int64_t n, S &&spill) {
        const Node &x = node[n];
        const bool tab = in_table(n);
        auto r_of = [&](int32_t c) { return (int)(tab ? need[c].t : need[c].g); };
        auto f_of = [&](int32_t c) { return (int)(tab ? need[c].fuse_t : need[c].fuse_g); };
        int r[3] = {r_of(x.k[0]), r_of(x.k[1]), r_of(x.k[2])};
        int best = 0, best_p = 0;
        for (;;) {
            int worst = 0;  // the most demanding child (the first one of several)
            if (x.op == TGP_WARP) {  // t0 then t1 on the stack, in that order
                best = std::max(r[1], 1 + r[2]);
                best_p = 0;
                worst = r[1] >= r[2] ? 1 : 2;
            } else if (x.ar < 3) {
                // (an absent child needs nothing and fuses nothing: the same
                // arithmetic serves every arity below three)
                const int f0 = (kOpForms.forward[x.op] >= 0) & f_of(x.k[1]);
                const int f1 = (kOpForms.backward[x.op] >= 0) & f_of(x.k[0]);
                const int v0 = std::max(r[0], f0 ? 0 : 1 + r[1]);
                const int v1 = std::max(r[1], f1 ? 0 : 1 + r[0]) | (x.ar == 2 && reorder ? 0 : 256);
                best = std::min(v0, v1);
                best_p = v1 < v0 ? 2 : 0;
                worst = r[1] > r[0] ? 1 : 0;
            } else {
                best = 1 << 30;
                for (int p = 0; p < (reorder ? 6 : 1); ++p) {
                    const uint8_t *o = kPerms[p];
                    const int v = std::max(r[o[0]], std::max(1 + r[o[1]], 2 + r[o[2]]));
                    if (v < best) {
                        best = v;
                        best_p = p;
                    }
                }
                for (int j = 1; j < 3; ++j)
                    if (r[j] > r[worst]) worst = j;
            }
            if (best <= D) break;
            const int32_t c = x.k[worst];
            spill(c);
            for (int j = 0; j < 3; ++j)
                if (x.k[j] == c) r[j] = 1;
        }
        best = x.ar == 0 ? 1 : best;
        perm[n] = (uint8_t)best_p;
        // as a child: a terminal or a value can be fused, a value takes one slot
        const bool value = in_table(n) || cached[n];
        const bool var = x.op == TGP_VAR && (split > 0 || axis(n) <= 1), cst = x.op == TGP_CONST;
        need[n] = Need{(uint8_t)(value ? 1 : best), (uint8_t)best, (uint8_t)(value || cst || (var && split == 0)),
                       (uint8_t)(cst || var)};
    }
    // Node c becomes a value: a cache row, or (in a table's own program) a
    // nested table entry.  Returns whether it was not one before.
    bool spill_node(int32_t c) {
        if (!in_table(c)) {
            need[c].g = 1;
            need[c].fuse_g = 1;
            return mark(cached, c);
        }
        mark(cached, c);
        need[c].t = 1;
        need[c].fuse_t = 1;
        return mark(nested, c);
    }

    // Whether caching node n, evaluated uses[n] times, pays for its traffic.
    bool pays(int64_t n) const {
        const double un = (double)uses[n];
        return un >= 2 && !cached[n] && access_cost >= 0 && node[n].ar > 0 && !in_table(n) &&
               cost[n] * (un - 1) > access_cost * (un + 1);
    }
    // How often node n evaluates each of its children.
    int64_t contribution(int64_t n) const { return pre[n] ? 0 : (cached[n] ? 1 : uses[n]); }
    // Fill level of node n, after the levels of its children.
    void up_level(int64_t n) {
        const Node &x = node[n];
        if (cached[n] && !pre[n] && uses[n] == 0) cached[n] = 0;  // a spill that nothing reads
        int32_t dp = 0;
        const std::vector<uint8_t> &value = in_table(n) ? nested : cached;
        for (int j = 0; j < 3; ++j) {
            const int32_t c = x.k[j];
            dp = std::max(dp, value[c] ? level[c] + 1 : dep[c]);
        }
        dep[n] = dp;
        level[n] = cached[n] && !pre[n] ? dp : -1;  // resident: available before the first level
    }

    // The same decisions made level by level (DAG node heights) on T host
    // threads.  Within a level the nodes are independent: each reads only
    // what lower levels decided (bottom-up passes) or higher levels
    // contributed (the top-down use counts), so the outcome does not depend
    // on thread timing.  It can differ from the sequential form in one way:
    // two parents of one height that share a child do not see each other's
    // stack spills, so both may spill where the sequential pass spilled
    // once.  Cache-budget admissions are made in node order within a level.
    tgp_status decide_parallel(const std::vector<int32_t> &rootrefs, std::string &why, int T) {
        const int64_t U = (int64_t)d.op.size();
        if (lorder.size() != (size_t)U) height_order(team, d.height.data(), U, T, lorder, lfirst);
        const std::vector<int32_t> &order = lorder;
        const int32_t H = (int32_t)lfirst.size() - 2;
        resize(U);
        std::vector<double> valu_part(T, 0.0);
        std::vector<std::vector<int32_t>> spill(T), cand(T);
        std::vector<std::array<int64_t, 3>> slot_part(T + 1);  // cache rows, row table, column table
        for (auto &c : slot_part) c.fill(0);
        std::vector<std::array<int64_t, 2>> tab_part(T);
        std::atomic<int64_t> used{0}, table_spills{0};
        std::atomic<bool> warps{false};
        const bool resident = !d.precached.empty() && access_cost >= 0;
        tgp_status result = TGP_OK;
        run_team(team, T, [&](int t, auto &barrier) {
            const int64_t b = U * t / T, e = U * (t + 1) / T;
            auto for_level = [&](int32_t h, auto &&fn) {
                const int64_t n0 = lfirst[h], n1 = lfirst[h + 1];
                for (int64_t i = n0 + (n1 - n0) * t / T; i < n0 + (n1 - n0) * (t + 1) / T; ++i) fn(order[i]);
            };
            double v = 0;
            bool w = false;
            for (int64_t n = b; n < e; ++n) {
                v += load(n, U);
                w |= node[n].op == TGP_WARP;
            }
            valu_part[t] = v;
            if (w) warps = true;
            barrier();
            const bool warp_first = warps;
            if (warp_first) {  // every cost, then the values warps gather from
                for (int32_t h = 0; h <= H; ++h) {
                    for_level(h, [&](int32_t n) { up_cost(n, resident, rootrefs[n] > 0); });
                    barrier();
                }
                int64_t u = 0;
                for (int64_t n = b; n < e; ++n)
                    if (node[n].op == TGP_WARP && mark(cached, node[n].k[0])) ++u;
                used.fetch_add(u);
                barrier();
            }
            // bottom-up; the spills of one level are applied after it
            for (int32_t h = 0; h <= H; ++h) {
                spill[t].clear();
                for_level(h, [&](int32_t n) {
                    if (!warp_first) up_cost(n, resident, rootrefs[n] > 0);
                    up_need(n, [&](int32_t c) { spill[t].push_back(c); });
                });
                barrier();
                int64_t su = 0, st = 0;
                for (int32_t c : spill[t])
                    if (spill_node(c)) ++(in_table(c) ? st : su);
                if (su) used.fetch_add(su);
                if (st) table_spills.fetch_add(st);
                barrier();
            }
            if (split > 0) {
                tab_part[t] = {0, 0};
                for (int64_t n = b; n < e; ++n)
                    if (cached[n] && in_table(n)) ++tab_part[t][cls[n] - 1];
                barrier();
            }
            if (t == 0) {
                spills = used.load() + table_spills.load();
                if (split > 0) {
                    int64_t entries[2] = {0, 0};
                    for (int i = 0; i < T; ++i)
                        for (int q = 0; q < 2; ++q) entries[q] += tab_part[i][q];
                    if (!set_table_slots(entries)) result = TGP_ENOMEM;
                    used.fetch_add((int64_t)table_slots);
                }
                if ((size_t)used.load() > budget_slots) {
                    tables_over = split > 0;
                    why = "the subtree cache needed to bound the evaluator stack exceeds the cache budget";
                    result = TGP_ENOMEM;
                }
            }
            // use counts, top-down; caching where it pays for its HBM traffic
            for (int64_t n = b; n < e; ++n) uses[n] = rootrefs[n];
            barrier();
            if (result != TGP_OK) return;
            for (int32_t h = H; h >= 0; --h) {
                cand[t].clear();
                for_level(h, [&](int32_t n) {
                    if (pays(n)) cand[t].push_back(n);
                });
                barrier();
                if (t == 0) {  // admissions in node order (within the budget)
                    for (int i = 0; i < T; ++i)
                        for (int32_t n : cand[i])
                            if ((size_t)used.load() < budget_slots) {
                                cached[n] = 1;
                                used.fetch_add(1);
                            }
                }
                barrier();
                // A count is at most the number of occurrences of the node in
                // the population's trees (each unit is one root-to-node path),
                // so it cannot overflow.  Leaves are skipped unless cached (a
                // warp source, a table entry): nothing reads their counts, and
                // they are the most shared nodes, so their additions would
                // contend most.
                for_level(h, [&](int32_t n) {
                    const int64_t contrib = contribution(n);
                    if (contrib > 0)
                        for (int j = 0; j < node[n].ar; ++j) {
                            const int32_t c = node[n].k[j];
                            if (node[c].ar > 0 || (cached[c] && __atomic_load_n(&uses[c], __ATOMIC_RELAXED) == 0))
                                __atomic_fetch_add(&uses[c], contrib, __ATOMIC_RELAXED);
                        }
                });
                barrier();
            }
            for (int32_t h = 0; h <= H; ++h) {
                for_level(h, [&](int32_t n) { up_level(n); });
                barrier();
            }
            // slots in node order
            std::array<int64_t, 3> cnt{0, 0, 0};
            for (int64_t n = b; n < e; ++n)
                if (cached[n]) ++cnt[in_table(n) ? cls[n] : 0];
            slot_part[t + 1] = cnt;
            barrier();
            std::array<int64_t, 3> ns{0, 0, 0};
            for (int i = 0; i <= t; ++i)
                for (int q = 0; q < 3; ++q) ns[q] += slot_part[i][q];
            for (int64_t n = b; n < e; ++n)
                if (cached[n]) slot[n] = (int32_t)ns[in_table(n) ? cls[n] : 0]++;
        });
        valu_dag = 0;
        for (double v : valu_part) valu_dag += v;
        trim(U);
        return result;
    }

    // Decide the cached nodes; returns TGP_OK or an error.
    tgp_status decide(const std::vector<int32_t> &rootrefs, std::string &why) {
        const int64_t U = (int64_t)d.op.size();
        resize(U);
        valu_dag = 0;
        bool warps = false;
        for (int64_t n = 0; n < U; ++n) {
            valu_dag += load(n, U);
            warps |= node[n].op == TGP_WARP;
        }
        const bool resident = !d.precached.empty() && access_cost >= 0;
        size_t used = 0;
        int64_t table_spills = 0;  // table entries only a table's own program needs
        // The value a warp gathers from is read at other cases than the one
        // being evaluated, so it is always materialised (a cached row), which
        // every other parent of it then reads.
        if (warps) {
            for (int64_t n = 0; n < U; ++n) up_cost(n, resident, rootrefs[n] > 0);
            for (int64_t n = 0; n < U; ++n)
                if (node[n].op == TGP_WARP && mark(cached, node[n].k[0])) ++used;
        }
        // Bottom-up (children have smaller ids).
        for (int64_t n = 0; n < U; ++n) {
            if (!warps) up_cost(n, resident, rootrefs[n] > 0);
            up_need(n, [&](int32_t c) {
                const bool fresh = spill_node(c);
                if (in_table(c)) table_spills += fresh;
                else used += fresh;
            });
        }
        spills = (int64_t)used + table_spills;
        if (split > 0) {
            int64_t entries[2] = {0, 0};
            for (int64_t n = 0; n < U; ++n)
                if (cached[n] && in_table(n)) ++entries[cls[n] - 1];
            if (!set_table_slots(entries)) return TGP_ENOMEM;
            used += table_slots;
        }
        if (used > budget_slots) {
            tables_over = split > 0;
            why = "the subtree cache needed to bound the evaluator stack exceeds the cache budget";
            return TGP_ENOMEM;
        }
        // Top-down: how often each node would be evaluated, and whether
        // caching it pays for its HBM traffic (within the remaining budget).
        for (int64_t n = 0; n < U; ++n) uses[n] = rootrefs[n];
        for (int64_t n = U - 1; n >= 0; --n) {
            if (pays(n) && used < budget_slots) {
                cached[n] = 1;
                ++used;
            }
            const int64_t contrib = contribution(n);
            const Node &x = node[n];
            uses[x.k[0]] += contrib;
            uses[x.k[1]] += contrib;
            uses[x.k[2]] += contrib;
        }
        // Levels and slots.
        int32_t ns[3] = {0, 0, 0};  // cache rows, row table, column table
        for (int64_t n = 0; n < U; ++n) {
            up_level(n);
            if (cached[n]) slot[n] = ns[in_table(n) ? cls[n] : 0]++;
        }
        trim(U);
        return TGP_OK;
    }

    // The FP32 bits of constant (or folded) node n; every NaN becomes the
    // quiet NaN 0x7fc00000, so that no signalling NaN reaches the
    // interpreter's min and max (ops_device.h).
    uint32_t const_word(int64_t n) const {
        const float v = !folded.empty() && folded[n] ? fold_val[n] : d.value[n];
        uint32_t w;
        memcpy(&w, &v, 4);
        return v == v ? w : 0x7fc00000u;
    }

    // The fused-form kind and .y word of child c when c can be a fused
    // operand (x, y, a constant or a cached row), else -1.
    // uc: the class of the program (3 unless it fills a table).
    int fuse_operand(int32_t c, uint32_t &y, int uc) const {
        if (uc == 3 ? cached[c] : nested[c]) {
            y = (uint32_t)slot[c];
            return uc == 3 && in_table(c) ? (cls[c] == 1 ? kFuseX : kFuseY) : kFuseCache;
        }
        const int o = op(c);
        if (o == TGP_VAR) {
            const int v = axis(c) - (uc == 2 ? split : 0);
            return v == 0 ? kFuseX : (v == 1 ? kFuseY : -1);
        }
        if (o == TGP_CONST) {
            y = const_word(c);
            return kFuseConst;
        }
        return -1;
    }

    // Postfix program of node n (n itself is expanded even when cached).
    // Every instruction carries the stack depth before it (.x bits 8-15).
    // A binary operator whose last-evaluated child is a terminal takes its
    // fused form and reads that child itself.  Adds the cost-model slots of
    // its instructions to *valu; sets *ext when it emits a bitwise operator,
    // warp or the third axis, *warp_used for warp.
    // The program of a table entry is a flat one over its own axes; with `ref`
    // a root that is a table entry is read from its table instead.
    void emit(int32_t root, std::vector<uint2> &code, int64_t &cache_reads, double *valu, bool *ext,
              bool *warp_used, bool ref) const {
        if (ref && in_table(root)) {
            code.push_back(uint2{cls[root] == 1 ? (uint32_t)I_X : (uint32_t)I_Y, (uint32_t)slot[root]});
            code.push_back(uint2{(1u << 8) | I_END, 0});
            *valu += 1.0;
            return;
        }
        const int uc = in_table(root) ? cls[root] : 3;
        auto value = [&](int32_t n) { return n != root && (uc == 3 ? cached[n] : nested[n]) != 0; };
        // An operator whose operands are being emitted: its stacked children
        // in evaluation order, and the operand its fused form reads itself.
        struct Frame {
            int32_t n;
            int32_t kid[3];
            uint8_t done, stacked;
            int8_t fv;         // fused form index, or -1
            uint8_t kind;      // fused operand kind
            uint32_t y;        // and its instruction word
            int32_t operand;   // and node
        };
        thread_local std::vector<Frame> st;
        st.clear();
        int64_t reads = 0;
        double slots = 0;
        uint32_t S = 0;  // stack depth before the next instruction
        auto put = [&](uint32_t c, uint32_t y) { code.push_back(uint2{c | S << 8, y}); };
        // a value read from a row or a terminal is one instruction; an
        // operator opens a frame
        auto open = [&](int32_t n) {
            if (value(n)) {
                const bool tab = uc == 3 && in_table(n);
                put(tab ? (cls[n] == 1 ? I_X : I_Y) : I_CACHE, (uint32_t)slot[n]);
                if (uc == 3 && !tab) ++reads;
                slots += 1.0;
                ++S;
                return;
            }
            const int o = op(n), a = arity(n);
            slots += kOpCost[o];
            if (a == 0) {
                if (o == TGP_VAR) {
                    const int v = axis(n) - (uc == 2 ? split : 0);
                    put(v == 0 ? I_X : (v == 1 ? I_Y : I_Z), 0);
                    if (v > 1) *ext = true;  // the third axis: extended interpreter only
                } else {
                    put(I_CONST, const_word(n));
                }
                ++S;
                return;
            }
            Frame f;
            f.n = n;
            f.done = 0;
            f.fv = -1;
            f.stacked = (uint8_t)a;
            const int32_t *k = node[n].k;
            if (o == TGP_WARP) {  // stack children t0, t1 only
                f.kid[0] = k[1];
                f.kid[1] = k[2];
                f.stacked = 2;
            } else {
                const uint8_t *order = kPerms[perm[n]];
                for (int j = 0; j < a; ++j) f.kid[j] = k[order[j]];
                if (a == 2) {
                    const int fv = order[1] ? kOpForms.forward[o] : kOpForms.backward[o];
                    uint32_t y = 0;
                    const int kind = fv >= 0 ? fuse_operand(f.kid[1], y, uc) : -1;
                    // two table values: a pair form
                    const int32_t c0 = f.kid[0];
                    if (kind >= 0 && uc == 3 && value(c0) && in_table(c0) && in_table(f.kid[1]) &&
                        cls[c0] != cls[f.kid[1]] && std::max(slot[c0], slot[f.kid[1]]) < 65536) {
                        // the row-table value is the first operand, unless it
                        // is child 1
                        const int32_t rc = cls[c0] == 1 ? c0 : f.kid[1], cc = cls[c0] == 1 ? f.kid[1] : c0;
                        const bool rev = k[0] != rc && !is_commutative(o);
                        put(kPairBase + (uint32_t)fused_index(o, rev), (uint32_t)slot[cc] << 16 | (uint32_t)slot[rc]);
                        slots += 2.0;
                        ++S;
                        return;
                    }
                    if (kind >= 0) {
                        f.fv = (int8_t)fv;
                        f.kind = (uint8_t)kind;
                        f.y = y;
                        f.operand = f.kid[1];
                        f.stacked = 1;
                    }
                }
            }
            st.push_back(f);
        };
        open(root);
        while (!st.empty()) {
            Frame &top = st.back();
            if (top.done < top.stacked) {
                open(top.kid[top.done++]);  // may move the frames
                continue;
            }
            const int32_t n = top.n;
            const int o = op(n);
            if (top.fv >= 0) {
                if (value(top.operand)) {
                    if (top.kind == kFuseCache && uc == 3) ++reads;
                    slots += 1.0;
                } else {
                    slots += kOpCost[op(top.operand)];
                }
                put(kFuseBase + 16 * (uint32_t)top.kind + (uint32_t)top.fv, top.y);
            } else if (o == TGP_OR || o == TGP_XOR || o == TGP_AND) {
                put(kFnBase + TGP_OR, (uint32_t)(o - TGP_OR));
                *ext = true;
                --S;
            } else if (o == TGP_WARP) {
                put(I_WARP, (uint32_t)slot[node[n].k[0]]);
                *ext = *warp_used = true;
                ++reads;
                --S;
            } else {
                const int a = kArity[o];
                if (perm[n] == 0 || (a == 2 && is_commutative(o))) put(kFnBase + o, 0);
                else if (a == 2) put(kRevBase + o, 0);
                else put(kPermBase + 6 * ternary_index(o) + perm[n], 0);
                S -= (uint32_t)a - 1;
            }
            st.pop_back();
        }
        code.push_back(uint2{(S << 8) | I_END, 0});
        cache_reads += reads;
        *valu += slots;
    }
};

}  // namespace

// (named in the context, so not in this file's own namespace)
struct PlanScratch {
    std::vector<uint8_t> cached, pre, perm, cls, nested;
    std::vector<int32_t> slot, level, lorder, dep;
    std::vector<double> cost;
    std::vector<int64_t> uses;
    std::vector<Planner::Node> node;
    std::vector<Planner::Need> need;
    std::vector<std::vector<uint2>> emitted;
};

namespace {

void Planner::swap_scratch(PlanScratch &o) {
    cached.swap(o.cached);
    pre.swap(o.pre);
    perm.swap(o.perm);
    cls.swap(o.cls);
    nested.swap(o.nested);
    slot.swap(o.slot);
    level.swap(o.level);
    lorder.swap(o.lorder);
    dep.swap(o.dep);
    cost.swap(o.cost);
    uses.swap(o.uses);
    node.swap(o.node);
    need.swap(o.need);
    emitted.swap(o.emitted);
    lorder.clear();
}

// Lends a context's arrays to the planner of one plan.
struct ScratchLoan {
    Planner &pl;
    PlanScratch &sc;
    ScratchLoan(tgp_ctx ctx, Planner &p) : pl(p), sc(get(ctx)) { pl.swap_scratch(sc); }
    ~ScratchLoan() { pl.swap_scratch(sc); }
    static PlanScratch &get(tgp_ctx ctx) {
        if (!ctx->plan_scratch) ctx->plan_scratch = std::make_shared<PlanScratch>();
        return *ctx->plan_scratch;
    }
};

// Programs of many nodes emitted by a few host threads (emission only reads
// the planner's decisions); each node's code stays contiguous, in order.
struct Emitted {
    uint32_t off, len;
    int64_t reads;
    double valu;
    bool ext, warp;  // uses the bitwise operators or warp
};

void emit_all(Planner &pl, const std::vector<int32_t> &nodes, std::vector<uint2> &code,
              std::vector<Emitted> &out, int threads, bool ref) {
    const size_t n = nodes.size();
    out.assign(n, Emitted{0, 0, 0, 0.0, false, false});
    // (a thread for every 128 programs; threads of its own only for 512)
    const int per = pl.team ? 128 : 512;
    const int T = team_size(
        pl.team, std::max(1, std::min({(int)(n / per) * (pl.team ? 1 : threads), threads, (int)usable_cpus()})));
    if (T == 1) {
        for (size_t i = 0; i < n; ++i) {
            Emitted &m = out[i];
            m.off = (uint32_t)code.size();
            pl.emit(nodes[i], code, m.reads, &m.valu, &m.ext, &m.warp, ref);
            m.len = (uint32_t)(code.size() - m.off);
        }
        return;
    }
    std::vector<std::vector<uint2>> &local = pl.emitted;
    if ((int)local.size() < T) local.resize(T);
    auto work = [&](int t) {
        const size_t b = n * t / T, e = n * (t + 1) / T;
        local[t].clear();
        for (size_t i = b; i < e; ++i) {
            Emitted &m = out[i];
            m.off = (uint32_t)local[t].size();
            pl.emit(nodes[i], local[t], m.reads, &m.valu, &m.ext, &m.warp, ref);
            m.len = (uint32_t)(local[t].size() - m.off);
        }
    };
    run_threads(pl.team, T, work);
    std::vector<uint32_t> base(T + 1, (uint32_t)code.size());
    for (int t = 0; t < T; ++t) base[t + 1] = base[t] + (uint32_t)local[t].size();
    code.resize(base[T]);
    run_threads(pl.team, T, [&](int t) {
        std::copy(local[t].begin(), local[t].end(), code.begin() + base[t]);
        for (size_t i = n * t / T; i < n * (t + 1) / T; ++i) out[i].off += base[t];
    });
}

}  // namespace

// ------------------------------------------------------------------ planning
// DAGs of at least this many nodes are planned level-parallel on host threads,
// at most kPlanThreads of them (fewer when the host has fewer processors).
constexpr int64_t kParallelDecideNodes = 1 << 15;
constexpr int kPlanThreads = 16;

//
// Planning one DAG runs in phases so that a batch of many DAGs can run each
// phase for all of them at once: host preparation (program lists, the
// variable-free subtrees), constant folding on the device (one round trip
// for the whole batch), the caching and stack decisions with program
// emission (host, one DAG per thread), and the upload of the programs (only
// for the single-DAG calls; a batch packs the host copies itself).
struct PlanJob {
    tgp_dag d;
    int64_t cases;
    Planner pl;
    std::vector<int32_t> rootrefs, ind_rows, store_of, store_list;
    std::vector<std::pair<int32_t, int32_t>> reduce_list;  // (root node, channel)
    // variable-free nodes by height (folding), this job's place in the batch
    std::vector<int32_t> fold_first, fold_list;
    size_t fold_list_at = 0, fold_val_at = 0;
    int64_t tab_rows = 0;  // grid rows of the domain at its split
    size_t budget = 0;     // cache budget in bytes
    double t_decide = 0, t_emit = 0;
    std::vector<uint2> code;  // becomes the plan's code
    // fill-program figures carried from the fill emission to the root one
    int64_t cache_reads_fill = 0;
    double valu_fill = 0;
    tgp_status st = TGP_OK;
    std::string err;
    PlanJob(tgp_dag dag, int64_t n_cases, int D, size_t budget)
        : d(dag), cases(n_cases), pl(*dag, D, budget) {}
};

static void plan_prepare(PlanJob &w, bool fold, int threads = 1) {
    tgp_dag d = w.d;
    Plan &P = d->plan;
    const int64_t U = d->stats.dag_nodes, R = d->stats.n_roots;
    const int n_ch = d->n_ch;
    // distinct programs
    std::unordered_map<int64_t, int32_t> reduce_of;  // (root id, ch) -> program
    w.rootrefs.assign(U, 0);
    w.ind_rows.resize(R);
    w.store_of.assign(U, -1);
    P.store_rows.assign(R, -1);
    P.dup_src.assign(R, -1);
    for (int64_t r = 0; r < R; ++r) {
        const int32_t n = d->roots[r];
        const int ch = (int)(r % n_ch);
        const int64_t key = (int64_t)n * n_ch + ch;
        auto it = reduce_of.find(key);
        if (it == reduce_of.end()) {
            it = reduce_of.emplace(key, (int32_t)w.reduce_list.size()).first;
            w.reduce_list.push_back({n, ch});
            w.rootrefs[n] += 1;
        }
        w.ind_rows[r] = it->second;
        if (w.store_of[n] < 0) {
            w.store_of[n] = (int32_t)r;
            w.store_list.push_back(n);
            P.store_rows[r] = (int32_t)r;
        } else {
            P.dup_src[r] = w.store_of[n];
        }
    }
    if (!fold) return;
    // Constant subtrees (no variable below) that some non-constant node or a
    // root uses are folded: marked in pl.folded, evaluated on the device.
    // novar: no variable below; 2 = also an operator (a foldable subtree)
    std::vector<uint8_t> novar(U, 0), use(U, 0);
    int64_t n_use = 0;
    auto mark = [&](int32_t c) {
        if (novar[c] == 2 && !use[c]) {
            use[c] = 1;
            ++n_use;
        }
    };
    const int32_t *kid = d->kid.data();
    const int32_t *height = d->height.data();
    int T = (int)std::min<unsigned>((unsigned)std::max(threads, 1), usable_cpus());
    if (U >= kParallelDecideNodes) T = team_size(w.pl.team, T);
    if (U >= kParallelDecideNodes && T > 1) {
        // level by level on T threads; the height order is kept for the
        // parallel decisions
        std::vector<int32_t> &order = w.pl.lorder;
        std::vector<int64_t> &first = w.pl.lfirst;
        height_order(w.pl.team, height, U, T, order, first);
        const int32_t H = (int32_t)first.size() - 2;
        std::atomic<int64_t> marked{0};
        run_team(w.pl.team, T, [&](int t, auto &barrier) {
            int64_t m = 0;
            for (int32_t h = 0; h <= H; ++h) {
                const int64_t n0 = first[h], n1 = first[h + 1];
                for (int64_t i = n0 + (n1 - n0) * t / T; i < n0 + (n1 - n0) * (t + 1) / T; ++i) {
                    const int32_t n = order[i];
                    const int o = d->op[n] & 0xff;
                    const int a = kArity[o];
                    bool nv = o != TGP_VAR;
                    for (int j = 0; j < a; ++j) nv = nv && novar[kid[3 * (int64_t)n + j]];
                    if (nv) {
                        novar[n] = a > 0 ? 2 : 1;
                    } else {
                        for (int j = 0; j < a; ++j) {
                            const int32_t c = kid[3 * (int64_t)n + j];
                            if (novar[c] == 2) {
                                __atomic_store_n(&use[c], (uint8_t)1, __ATOMIC_RELAXED);
                                ++m;
                            }
                        }
                    }
                }
                barrier();
            }
            marked.fetch_add(m);
        });
        n_use = marked.load();
        for (int32_t r : d->roots) mark(r);
        if (n_use == 0) return;
        w.fold_first.assign(1, 0);
        for (int32_t h = 0; h <= H; ++h) {
            for (int64_t i = first[h]; i < first[h + 1]; ++i)
                if (novar[order[i]] == 2) w.fold_list.push_back(order[i]);
            w.fold_first.push_back((int32_t)w.fold_list.size());
        }
        // up to the highest variable-free operator node
        while (w.fold_first.size() > 1 && w.fold_first[w.fold_first.size() - 2] == w.fold_first.back())
            w.fold_first.pop_back();
        w.pl.folded.swap(use);
        return;
    }
    // the variable-free operator nodes by height (constant leaves are read
    // from the node values by the fold kernel)
    std::vector<std::vector<int32_t>> by_h;
    for (int64_t n = 0; n < U; ++n) {  // children have smaller ids
        const int o = d->op[n] & 0xff;
        const int a = kArity[o];
        bool nv = o != TGP_VAR;
        for (int j = 0; j < a; ++j) nv = nv && novar[kid[3 * n + j]];
        if (nv) {
            novar[n] = a > 0 ? 2 : 1;
            if (a > 0) {
                const int32_t h = height[n];
                if ((int32_t)by_h.size() <= h) by_h.resize(h + 1);
                by_h[h].push_back((int32_t)n);
            }
        } else {
            for (int j = 0; j < a; ++j) mark(kid[3 * n + j]);
        }
    }
    for (int32_t r : d->roots) mark(r);
    if (n_use == 0) return;
    // children before parents: one list, cut at each height
    w.fold_first.assign(by_h.size() + 1, 0);
    for (size_t h = 0; h < by_h.size(); ++h) w.fold_first[h + 1] = w.fold_first[h] + (int32_t)by_h[h].size();
    w.fold_list.reserve(w.fold_first.back());
    for (const auto &v : by_h) w.fold_list.insert(w.fold_list.end(), v.begin(), v.end());
    w.pl.folded.swap(use);
}

// Folds one job's marked subtrees in one launch that reads the node list from,
// and writes the values to, the pinned staging.
static hipError_t fold_one(tgp_ctx ctx, PlanJob &w) {
    const int32_t n = (int32_t)w.fold_list.size(), heights = (int32_t)w.fold_first.size() - 1;
    const int64_t U = w.d->stats.dag_nodes;
    void *pos = nullptr, *stage = nullptr;
    hipError_t e = ctx->pool.alloc(&pos, sizeof(int32_t) * U);
    if (e == hipSuccess) e = ctx_pinned(ctx, sizeof(int32_t) * (2 * (size_t)n + heights + 1), &stage);
    if (e == hipSuccess) {
        int32_t *list = static_cast<int32_t *>(stage), *first = list + n;
        float *out = reinterpret_cast<float *>(first + heights + 1);
        memcpy(list, w.fold_list.data(), sizeof(int32_t) * n);
        memcpy(first, w.fold_first.data(), sizeof(int32_t) * (heights + 1));
        e = launch_fold_all(FoldDesc{w.d->dev.node_op, w.d->dev.node_value, w.d->dev.node_kid, static_cast<float *>(pos)},
                            list, n, first, heights, out, ctx->stream);
        const hipError_t es = hipStreamSynchronize(ctx->stream);
        if (e == hipSuccess) e = es;
        if (e == hipSuccess) {
            w.pl.fold_val.resize(U);
            for (int32_t i = 0; i < n; ++i) w.pl.fold_val[w.fold_list[i]] = out[i];
        }
    }
    ctx->pool.release(pos);
    return e;
}

// Folds the marked subtrees of every job.  A single DAG's few nodes: one
// launch (fold_one).  Otherwise one upload of the node lists, one launch per
// height over all jobs, one read-back of the values.
static tgp_status fold_run(tgp_ctx ctx, const std::vector<PlanJob *> &jobs) {
    std::vector<PlanJob *> fj;
    size_t n_list = 0, n_val = 0;
    int32_t max_h = -1;
    for (PlanJob *w : jobs)
        if (!w->fold_list.empty()) {
            w->fold_list_at = n_list;
            w->fold_val_at = n_val;
            n_list += w->fold_list.size();
            n_val += (size_t)w->d->stats.dag_nodes;
            max_h = std::max(max_h, (int32_t)w->fold_first.size() - 2);
            fj.push_back(w);
        }
    if (fj.empty()) return TGP_OK;
    if (fj.size() == 1 && n_list <= (size_t)kFoldNodes && max_h < kFoldHeights) {
        const hipError_t e1 = fold_one(ctx, *fj[0]);
        if (e1 != hipSuccess) return fail(ctx, TGP_EHIP, "constant folding: %s", hipGetErrorString(e1));
        return TGP_OK;
    }
    // the (job, node) lists of all jobs ordered by height, then job
    std::vector<int32_t> hfirst(max_h + 2, 0);
    for (PlanJob *w : fj)
        for (size_t h = 0; h + 1 < w->fold_first.size(); ++h)
            hfirst[h + 1] += w->fold_first[h + 1] - w->fold_first[h];
    for (int h = 0; h <= max_h; ++h) hfirst[h + 1] += hfirst[h];
    const size_t desc_bytes = sizeof(FoldDesc) * fj.size();
    const size_t list_off = (desc_bytes + 255) & ~(size_t)255;
    const size_t val_off = (list_off + sizeof(int2) * n_list + 255) & ~(size_t)255;
    const size_t up_bytes = list_off + sizeof(int2) * n_list;
    void *blk = nullptr, *stage = nullptr;
    hipError_t e = ctx->pool.alloc(&blk, val_off + sizeof(float) * n_val);
    if (e == hipSuccess) e = ctx_pinned(ctx, std::max(up_bytes, sizeof(float) * n_val), &stage);
    if (e == hipSuccess) {
        FoldDesc *desc = static_cast<FoldDesc *>(stage);
        int2 *list = reinterpret_cast<int2 *>(static_cast<char *>(stage) + list_off);
        float *val_dev = reinterpret_cast<float *>(static_cast<char *>(blk) + val_off);
        std::vector<int32_t> at(hfirst.begin(), hfirst.end() - 1);
        for (size_t j = 0; j < fj.size(); ++j) {
            const PlanJob &w = *fj[j];
            desc[j] = FoldDesc{w.d->dev.node_op, w.d->dev.node_value, w.d->dev.node_kid, val_dev + w.fold_val_at};
            for (size_t h = 0; h + 1 < w.fold_first.size(); ++h)
                for (int32_t q = w.fold_first[h]; q < w.fold_first[h + 1]; ++q)
                    list[at[h]++] = int2{(int32_t)j, w.fold_list[q]};
        }
        e = hipMemcpyAsync(blk, stage, up_bytes, hipMemcpyHostToDevice, ctx->stream);
    }
    if (e == hipSuccess) e = ctx_pinned_enqueued(ctx);
    const FoldDesc *desc_dev = static_cast<const FoldDesc *>(blk);
    const int2 *list_dev = reinterpret_cast<const int2 *>(static_cast<char *>(blk) + list_off);
    for (int h = 0; h <= max_h && e == hipSuccess; ++h)
        e = launch_fold_level(desc_dev, list_dev + hfirst[h], hfirst[h + 1] - hfirst[h], ctx->stream);
    if (e == hipSuccess) e = ctx_pinned(ctx, sizeof(float) * n_val, &stage);
    if (e == hipSuccess)
        e = hipMemcpyAsync(stage, static_cast<char *>(blk) + val_off, sizeof(float) * n_val,
                           hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e == hipSuccess)
        for (PlanJob *w : fj) {
            const float *v = static_cast<const float *>(stage) + w->fold_val_at;
            w->pl.fold_val.assign(v, v + w->d->stats.dag_nodes);
        }
    hipStreamSynchronize(ctx->stream);
    ctx->pool.release(blk);
    if (e != hipSuccess) return fail(ctx, TGP_EHIP, "constant folding: %s", hipGetErrorString(e));
    return TGP_OK;
}

static void longest_first(std::vector<ProgDesc> &v) {
    std::stable_sort(v.begin(), v.end(), [](const ProgDesc &a, const ProgDesc &b) { return a.len > b.len; });
}

// Caching and stack decisions, then the fill programs by level (the first
// part of code_host).  Host only; emit_threads host threads emit.
static tgp_status plan_decide_emit_fill(PlanJob &w, int D, bool reorder, double access_cost, int fold,
                                        int emit_threads) {
    tgp_dag d = w.d;
    Plan &P = d->plan;
    Planner &pl = w.pl;
    const int64_t U = d->stats.dag_nodes;
    const double t0 = now_ms();
    P.n_folded = 0;
    for (uint8_t f : pl.folded) P.n_folded += f;
    pl.reorder = reorder;
    pl.access_cost = access_cost;
    const unsigned hw = usable_cpus();
    int dt = (int)std::min<unsigned>((unsigned)std::max(emit_threads, 1), hw);
    if (U >= kParallelDecideNodes) dt = team_size(pl.team, dt);
    auto decide = [&]() {
        return U >= kParallelDecideNodes && dt > 1 ? pl.decide_parallel(w.rootrefs, w.err, dt)
                                                   : pl.decide(w.rootrefs, w.err);
    };
    P.asked = pl.split;
    P.budget = w.budget;
    tgp_status st = decide();
    if (st != TGP_OK && pl.tables_over) {  // no room for the tables: flat programs
        size_t unused;
        const bool fit = tables_fit(pl.table_entries, pl.table_slots_per, pl.slot_bytes, pl.budget_slots, &unused);
        // (tables that fit, but not beside the rows that bound the stack: no shape has room for both)
        for (int q = 0; q < 2; ++q) P.refused[q] = fit ? INT32_MAX : pl.table_entries[q];
        if (d->other.cases >= 0) return TGP_ENOMEM;  // the flat plan is there already
        pl.split = 0;
        pl.tables_over = false;
        w.err.clear();
        st = decide();
    }
    if (st != TGP_OK) return st;
    P.split = pl.split;
    P.tab_rows = w.tab_rows;
    const double t1 = now_ms();
    w.t_decide = t1 - t0;

    std::vector<uint2> &code = w.code;
    std::vector<ProgDesc> fill;
    int32_t max_level = -1;
    std::vector<int32_t> cached_nodes, tab_nodes[2];
    int32_t max_tab = -1;
    for (int64_t n = 0; n < U; ++n)
        if (pl.cached[n]) {
            if (pl.in_table(n)) {
                tab_nodes[pl.cls[n] - 1].push_back((int32_t)n);
                max_tab = std::max(max_tab, pl.level[n]);
                continue;
            }
            cached_nodes.push_back((int32_t)n);
            max_level = std::max(max_level, pl.level[n]);
        }
    // the tables' programs, by level, row table first
    P.tab_host.clear();
    P.tab_level.assign(max_tab + 1, Plan::TabLevel{0, 0, 0});
    P.exec_tab[0] = P.exec_tab[1] = 0;
    std::vector<Emitted> em_tab;
    if (max_tab >= 0) {
        std::vector<int32_t> nodes(tab_nodes[0]);
        nodes.insert(nodes.end(), tab_nodes[1].begin(), tab_nodes[1].end());
        emit_all(pl, nodes, code, em_tab, emit_threads, false);
        std::vector<std::vector<ProgDesc>> part(2 * (size_t)(max_tab + 1));
        for (size_t i = 0; i < nodes.size(); ++i) {
            const int which = i < tab_nodes[0].size() ? 0 : 1;
            part[2 * (size_t)pl.level[nodes[i]] + which].push_back(
                ProgDesc{em_tab[i].off, em_tab[i].len, pl.slot[nodes[i]], 0});
            P.exec_tab[which] += em_tab[i].len - 1;
        }
        for (int32_t l = 0; l <= max_tab; ++l) {
            Plan::TabLevel &t = P.tab_level[l];
            t.first = (int32_t)P.tab_host.size();
            for (int which = 0; which < 2; ++which) {
                auto &v = part[2 * (size_t)l + which];
                longest_first(v);
                P.tab_host.insert(P.tab_host.end(), v.begin(), v.end());
                (which ? t.last : t.mid) = (int32_t)P.tab_host.size();
            }
        }
    }
    P.tab_code_end = (int64_t)code.size();
    for (int which = 0; which < 2; ++which) P.n_tab[which] = (int32_t)tab_nodes[which].size();
    P.slot_node.assign(cached_nodes.size(), -1);
    P.slot_pre.assign(cached_nodes.size(), 0);
    for (int32_t n : cached_nodes) {
        P.slot_node[pl.slot[n]] = n;
        P.slot_pre[pl.slot[n]] = pl.pre[n];
    }
    P.level_first.assign(max_level + 2, 0);
    std::vector<std::vector<ProgDesc>> by_level(max_level + 1);
    int64_t cache_reads_fill = 0;
    double valu_fill = 0;
    std::vector<int32_t> fill_nodes;
    for (int32_t n : cached_nodes)
        if (!pl.pre[n]) fill_nodes.push_back(n);
    std::vector<Emitted> em;
    emit_all(pl, fill_nodes, code, em, emit_threads, false);
    for (size_t i = 0; i < fill_nodes.size(); ++i) {
        const int32_t n = fill_nodes[i];
        ProgDesc pd{em[i].off, em[i].len, pl.slot[n], 0};
        cache_reads_fill += em[i].reads;
        valu_fill += em[i].valu;
        by_level[pl.level[n]].push_back(pd);
    }
    for (int l = 0; l <= max_level; ++l) {
        longest_first(by_level[l]);
        P.level_first[l] = (int32_t)fill.size();
        fill.insert(fill.end(), by_level[l].begin(), by_level[l].end());
    }
    P.level_first[max_level + 1] = (int32_t)fill.size();
    code.push_back(uint2{I_END, 0});  // padding past the last program
    P.D = D;
    P.reorder = reorder;
    P.access_cost = access_cost;
    P.fold = fold;
    P.ext = P.warp = false;
    for (const Emitted &m : em) {
        P.ext = P.ext || m.ext;
        P.warp = P.warp || m.warp;
    }
    P.n_slots = (int32_t)cached_nodes.size();
    P.n_spills = pl.spills;
    P.n_fill = (int32_t)fill.size();
    P.code_host = std::move(code);
    P.fill_host = std::move(fill);
    P.root_code_at = (int64_t)P.code_host.size();
    w.cache_reads_fill = cache_reads_fill;
    w.valu_fill = valu_fill;
    w.t_emit = now_ms() - t1;
    return TGP_OK;
}

// The root programs, appended to code_host: one per distinct (root,
// channel) for the fitness form and one per distinct root for the evaluate
// form.  Completes the plan.
static void plan_emit_roots(PlanJob &w, int emit_threads) {
    const double t0 = now_ms();
    Plan &P = w.d->plan;
    Planner &pl = w.pl;
    std::vector<uint2> &code = P.code_host;
    std::vector<ProgDesc> reduce, store;
    std::vector<Emitted> em;
    int64_t cache_reads_roots = 0;
    double exec_roots = 0;
    emit_all(pl, w.store_list, code, em, emit_threads, true);
    // program of each distinct root: store_list[i] <-> em[i], found through
    // the root's first row
    std::vector<int32_t> prog_of(w.d->roots.size(), -1);
    for (size_t i = 0; i < w.store_list.size(); ++i) prog_of[w.store_of[w.store_list[i]]] = (int32_t)i;
    double valu_roots = 0;
    for (size_t p = 0; p < w.reduce_list.size(); ++p) {
        const Emitted &m = em[prog_of[w.store_of[w.reduce_list[p].first]]];
        ProgDesc pd{m.off, m.len, (int32_t)p, w.reduce_list[p].second};
        reduce.push_back(pd);
        exec_roots += m.len - 1;
        cache_reads_roots += m.reads;
        valu_roots += m.valu;
    }
    for (size_t i = 0; i < w.store_list.size(); ++i) {
        ProgDesc pd{em[i].off, em[i].len, w.store_of[w.store_list[i]], 0};
        store.push_back(pd);
    }
    // reduce programs keep dest = their row; order them longest first
    longest_first(reduce);
    longest_first(store);
    code.push_back(uint2{I_END, 0});  // padding

    double exec_fill = 0;
    for (auto &pd : P.fill_host) exec_fill += pd.len - 1;
    P.exec_per_case = exec_fill + exec_roots;
    P.valu_dag_per_case = pl.valu_dag;
    P.valu_fill_per_case = w.valu_fill;
    P.valu_roots_per_case = valu_roots;
    P.cache_reads_per_case = w.cache_reads_fill + cache_reads_roots;
    P.instructions = (int64_t)code.size();
    for (const Emitted &m : em) {
        P.ext = P.ext || m.ext;
        P.warp = P.warp || m.warp;
    }
    P.n_reduce = (int32_t)reduce.size();
    P.n_store = (int32_t)store.size();
    P.reduce_host = std::move(reduce);
    P.store_host = std::move(store);
    P.ind_rows_host = std::move(w.ind_rows);
    P.cases = w.cases;
    if (P.split && w.d->ctx && w.d->ctx->plan_upload) P.fold_val.swap(w.pl.fold_val);
    w.t_emit += now_ms() - t0;
}

static tgp_status plan_decide_emit(PlanJob &w, int D, bool reorder, double access_cost, int fold,
                                   int emit_threads) {
    tgp_status st = plan_decide_emit_fill(w, D, reorder, access_cost, fold, emit_threads);
    if (st == TGP_OK) plan_emit_roots(w, emit_threads);
    return st;
}

// Bytes of a flat plan's programs in one block, 256-byte aligned parts.
static size_t flat_bytes(const Plan &P) {
    auto up = [](size_t n) { return (n + 255) & ~(size_t)255; };
    return up(sizeof(uint2) * P.code_host.size()) + up(sizeof(ProgDesc) * P.fill_host.size()) +
           up(sizeof(ProgDesc) * P.reduce_host.size()) + up(sizeof(ProgDesc) * P.store_host.size()) +
           up(sizeof(int32_t) * P.ind_rows_host.size());
}

// What a flat plan of d that tgp_fitness_noalloc can run needs at the most: a
// cached subtree's program stands where one occurrence of it was in the trees,
// which is a read now, so the code is no longer than the population's tokens
// with a read and an end for every row, and an end for every root; and only
// rows that fit the scratch count.
static size_t flat_bytes_bound(const tgp_dag_s &d, int64_t cases) {
    const size_t R = (size_t)d.stats.n_roots,
                 rows = (size_t)std::min<int64_t>(d.stats.dag_internal, kNoAllocScratchBytes / (4 * std::max<int64_t>(cases, 1)));
    return sizeof(uint2) * ((size_t)d.stats.tree_nodes + 2 * rows + R + 2) + sizeof(ProgDesc) * (rows + 2 * R) +
           sizeof(int32_t) * R + 5 * 256;
}

// Copies n parts into one new pool block (256-byte aligned parts) by one copy
// from the pinned staging; later launches on the stream see it in order.
// A part's `rebase`, when nonzero, is subtracted from the code offset of
// each of its ProgDesc entries as it is staged.
struct UploadPart {
    const void *src;
    size_t bytes;
    uint32_t rebase;
};
// The block has `spare` bytes behind the parts, from *base + off[n] on.
static hipError_t upload_parts(tgp_ctx ctx, int n, const UploadPart *part, void **blob, char **base,
                               size_t *off, size_t spare = 0) {
    size_t total = 0;
    for (int i = 0; i < n; ++i) {
        off[i] = total;
        total += (part[i].bytes + 255) & ~(size_t)255;
    }
    total = std::max<size_t>(total, 256);
    off[n] = total;
    void *stage = nullptr;
    hipError_t e = ctx->pool.alloc(blob, total + spare);
    if (e == hipSuccess) e = ctx_pinned(ctx, total, &stage);
    if (e != hipSuccess) return e;
    for (int i = 0; i < n; ++i) {
        if (!part[i].bytes) continue;
        char *dst = (char *)stage + off[i];
        memcpy(dst, part[i].src, part[i].bytes);
        if (part[i].rebase) {
            ProgDesc *pd = reinterpret_cast<ProgDesc *>(dst);
            for (size_t k = 0; k < part[i].bytes / sizeof(ProgDesc); ++k) pd[k].code_off -= part[i].rebase;
        }
    }
    e = hipMemcpyAsync(*blob, stage, total, hipMemcpyHostToDevice, ctx->stream);
    if (e == hipSuccess) e = ctx_pinned_enqueued(ctx);
    *base = static_cast<char *>(*blob);
    return e;
}

// The fill programs: code_host up to root_code_at and the fill descriptors.
static tgp_status plan_upload_fill(tgp_ctx ctx, Plan &P) {
    const UploadPart part[3] = {{P.code_host.data(), sizeof(uint2) * (size_t)P.root_code_at, 0},
                                {P.fill_host.data(), sizeof(ProgDesc) * P.fill_host.size(), 0},
                                {P.tab_host.data(), sizeof(ProgDesc) * P.tab_host.size(), 0}};
    size_t off[4];
    char *b = nullptr;
    hipError_t e = upload_parts(ctx, 3, part, &P.blob, &b, off);
    if (e != hipSuccess) {
        hipStreamSynchronize(ctx->stream);
        P.release(ctx->pool);
        return fail(ctx, TGP_EHIP, "plan upload: %s", hipGetErrorString(e));
    }
    P.code_dev = reinterpret_cast<uint2 *>(b + off[0]);
    P.fill_dev = reinterpret_cast<ProgDesc *>(b + off[1]);
    P.tab_dev = reinterpret_cast<ProgDesc *>(b + off[2]);
    return TGP_OK;
}

// The root programs: the rest of code_host, the reduce and store descriptors
// (offsets rebased to the start of that code) and the individual rows.
static tgp_status plan_upload_roots(tgp_ctx ctx, tgp_dag d, Plan &P) {
    const uint32_t at = (uint32_t)P.root_code_at;
    const UploadPart part[4] = {
        {P.code_host.data() + at, sizeof(uint2) * (P.code_host.size() - at), 0},
        {P.reduce_host.data(), sizeof(ProgDesc) * P.reduce_host.size(), at},
        {P.store_host.data(), sizeof(ProgDesc) * P.store_host.size(), at},
        {P.ind_rows_host.data(), sizeof(int32_t) * P.ind_rows_host.size(), 0}};
    size_t off[5];
    char *b = nullptr;
    P.reserve_bytes = P.split && !d->other.blob ? flat_bytes_bound(*d, P.cases) : 0;
    hipError_t e = upload_parts(ctx, 4, part, &P.blob_roots, &b, off, P.reserve_bytes);
    if (e != hipSuccess) {
        hipStreamSynchronize(ctx->stream);
        P.release(ctx->pool);
        return fail(ctx, TGP_EHIP, "plan upload: %s", hipGetErrorString(e));
    }
    P.code_roots_dev = reinterpret_cast<uint2 *>(b + off[0]);
    P.reduce_dev = reinterpret_cast<ProgDesc *>(b + off[1]);
    P.store_dev = reinterpret_cast<ProgDesc *>(b + off[2]);
    P.ind_rows_dev = reinterpret_cast<int32_t *>(b + off[3]);
    // Memory for tgp_fitness_noalloc alone.
    if (P.reserve_bytes) P.reserve = b + off[4];
    if (P.split) {
        const size_t rows = sizeof(float) * (size_t)P.n_slots * (size_t)P.cases, tables = P.planned_tables_bytes();
        const size_t sums = sizeof(float2) * (size_t)P.n_reduce * (size_t)((P.cases + kWideCols - 1) / kWideCols);
        if (rows <= kNoAllocScratchBytes && sums + rows + tables + 512 > kNoAllocScratchBytes &&
            ctx->pool.alloc(&P.noalloc_tables, tables) != hipSuccess) {  // (it may then refuse a call)
            P.noalloc_tables = nullptr;
            (void)hipGetLastError();
        }
    }
    return TGP_OK;
}

static tgp_status plan_upload(tgp_ctx ctx, tgp_dag d, Plan &P) {
    tgp_status st = plan_upload_fill(ctx, P);
    return st == TGP_OK ? plan_upload_roots(ctx, d, P) : st;
}

// Some words passed as a kernel argument.  One workgroup and 3840 bytes a launch
// (an argument block holds 4 KB), 2.5 us each: the programs of 176 trees, 1582
// words of code, take six, in a first call that plans for 0.1 ms as well.
struct PutWords {
    uint32_t w[960];
};
__global__ void k_put(const PutWords a, uint32_t *dst, int32_t n) {
    typedef const __attribute__((address_space(4))) uint32_t cword;
    const cword *src = (const cword *)__builtin_amdgcn_kernarg_segment_ptr();
    for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = src[i];
}

// Writes the blob of a flat plan made by flat_in_reserve: its words travel as
// kernel arguments, which needs no staging that would have to outlive a
// capture.  A captured call writes it where it is replayed, so the next call
// writes it again.
static tgp_status put_flat(tgp_ctx ctx, Plan &P) {
    if (!P.put) return TGP_OK;
    std::vector<char> image(flat_bytes(P));
    auto part = [&](const void *to, const void *src, size_t bytes) {
        if (bytes) memcpy(image.data() + ((const char *)to - (const char *)P.blob), src, bytes);
    };
    part(P.code_dev, P.code_host.data(), sizeof(uint2) * P.code_host.size());
    part(P.fill_dev, P.fill_host.data(), sizeof(ProgDesc) * P.fill_host.size());
    part(P.reduce_dev, P.reduce_host.data(), sizeof(ProgDesc) * P.reduce_host.size());
    part(P.store_dev, P.store_host.data(), sizeof(ProgDesc) * P.store_host.size());
    part(P.ind_rows_dev, P.ind_rows_host.data(), sizeof(int32_t) * P.ind_rows_host.size());
    hipStreamCaptureStatus cap = hipStreamCaptureStatusActive;
    if (hipStreamIsCapturing(ctx->stream, &cap) != hipSuccess) (void)hipGetLastError();
    for (size_t at = 0; at < image.size(); at += sizeof(PutWords)) {
        PutWords a;
        const size_t n = std::min(sizeof a, image.size() - at);
        memcpy(a.w, image.data() + at, n);
        hipLaunchKernelGGL(k_put, dim3(1), dim3(256), 0, ctx->stream, a, (uint32_t *)((char *)P.blob + at),
                           (int32_t)(n / 4));
    }
    HCHK(ctx, hipGetLastError());
    P.put = cap != hipStreamCaptureStatusNone;
    return TGP_OK;
}

int ctx_stack_slots(tgp_ctx ctx) { return ctx->stack_lds ? interp_lds_stack() : interp_max_stack(); }

// The split that d's programs get on dom under the context's settings: a
// chosen two cases per lane, the LDS stack, "no caching" (a negative access
// cost), unfolded constants, the image operators and very small work keep flat
// programs.
static int32_t wanted_split(tgp_ctx ctx, tgp_dag d, tgp_domain dom) {
    if (ctx->stack_lds || ctx->force_K == 2 || ctx->cache_access_cost < 0 || !ctx->fold) return 0;
    if (d->image_ops || d->no_tables) return 0;
    if (d->stats.dag_nodes < kTableNodes && d->stats.dag_nodes * dom->cases <= kTableWork) return 0;
    return dom->split;
}

// Cache slots of an entry of either table on dom split at `split`.
static void table_slots_on(tgp_domain dom, int32_t split, double (&per)[2]) {
    const double slot_bytes = sizeof(float) * (double)dom->cases;
    per[0] = (double)row_table_stride(*dom, split) / slot_bytes;
    per[1] = (double)col_table_stride(*dom, split) / slot_bytes;
}

// Gives the planner of w the split `split` of dom.
static void set_split(PlanJob &w, tgp_domain dom, int32_t split) {
    w.pl.split = split;
    if (!split) return;
    w.tab_rows = dom->rows(split);
    w.pl.slot_bytes = sizeof(float) * (double)dom->cases;
    table_slots_on(dom, split, w.pl.table_slots_per);
}

// Whether P was made for this number of cases and the context's settings.  A
// flat plan's programs run on any such domain, a plan's with tables where the
// tables fit (best_plan).
static bool plan_current(tgp_ctx ctx, const Plan &P, int64_t cases) {
    return P.cases == cases && P.D == ctx_stack_slots(ctx) && P.reorder == (ctx->reorder != 0) &&
           P.access_cost == ctx->cache_access_cost && P.fold == ctx->fold;
}

// Cache rows of `cases` cases in a budget of so many bytes.
static size_t rows_in(size_t budget, int64_t cases) {
    return (size_t)(budget / (sizeof(float) * (size_t)std::max<int64_t>(cases, 1)));
}

static bool tables_fit_on(size_t budget, const int64_t (&entries)[2], tgp_domain dom, int32_t split) {
    double per[2];
    size_t slots;
    table_slots_on(dom, split, per);
    return tables_fit(entries, per, sizeof(float) * (double)dom->cases, rows_in(budget, dom->cases), &slots);
}

// Of d's plans for domains of dom's size, the one to evaluate dom with, or
// nullptr if that one is not made yet: the one with tables where dom wants
// them (want, its split) and they fit, else the flat one.  The tables' size
// follows the grid's shape: a plan made on 1024 x 1024 cases may need hundreds
// of times as much on 8 x 131072, more than the budget and more than their
// 32-bit byte offsets reach.  On the shape that they were admitted for they
// stay as they were planned, like the cache rows.  *tables: which one it is.
static Plan *best_plan(tgp_ctx ctx, tgp_dag d, tgp_domain dom, int32_t want, bool *tables) {
    Plan *with = nullptr, *flat = nullptr;
    for (Plan *P : {&d->plan, &d->other})
        if (plan_current(ctx, *P, dom->cases)) (P->split ? with : flat) = P;
    *tables = want > 0;
    if (want > 0 && with) {
        const int64_t entries[2] = {with->n_tab[0], with->n_tab[1]};
        *tables = with->planned_shape(*dom) || tables_fit_on(with->budget, entries, dom, with->split);
    } else if (want > 0 && flat && flat->asked) {
        *tables = tables_fit_on(flat->budget, flat->refused, dom, flat->asked);
    }
    return *tables ? with : flat;
}

// Makes the plan to evaluate dom with d's plan in use.  *made: whether it is
// there; if not, d->plan is empty and *split says what to make (0: a flat plan).
// The other plan for the same size and settings is kept, so a DAG that is
// evaluated on several shapes of one size in turn is planned twice at most.
static tgp_status choose_plan(tgp_ctx ctx, tgp_dag d, tgp_domain dom, int32_t want, bool *made, int32_t *split) {
    bool tables;
    Plan *P = best_plan(ctx, d, dom, want, &tables);
    *made = P != nullptr;
    *split = tables ? want : 0;
    if (P) {
        if (P != &d->plan) std::swap(d->plan, d->other);
        return TGP_OK;
    }
    if (plan_current(ctx, d->plan, dom->cases)) std::swap(d->plan, d->other);
    for (Plan *Q : {&d->plan, &d->other})
        if (!plan_current(ctx, *Q, dom->cases) && !Q->store_rows.empty()) {  // (not a new DAG's)
            if (Q->blob) HCHK(ctx, hipStreamSynchronize(ctx->stream));  // no queued kernel reads it any more
            Q->release(ctx->pool);
            *Q = Plan();
        }
    return TGP_OK;
}

void forget_plans(tgp_ctx ctx, tgp_dag d) {
    for (Plan *P : {&d->plan, &d->other}) {
        P->release(ctx->pool);
        *P = Plan();
    }
}

// The cache budget of a plan made now: its neighbour's, so that a budget that was
// set for the DAG's first plan holds for every shape of its size.
static size_t plan_budget(tgp_ctx ctx, tgp_dag d) { return d->other.cases >= 0 ? d->other.budget : ctx->cache_budget; }

// After tables could not be planned beside a flat plan: goes on with the flat
// plan, for every shape (so that no call plans in vain again).
static void keep_flat(tgp_dag d) {
    std::swap(d->plan, d->other);
    d->plan.asked = d->other.asked;
    for (int64_t &n : d->plan.refused) n = INT32_MAX;
    d->other = Plan();
}

tgp_status build_plan(tgp_ctx ctx, tgp_dag d, tgp_domain dom, const std::function<tgp_status()> &after_fill) {
    const double t0 = now_ms();
    Plan &P = d->plan;
    const int64_t cases = dom->cases;
    int32_t split = 0;
    bool made = false;
    tgp_status st = choose_plan(ctx, d, dom, wanted_split(ctx, d, dom), &made, &split);
    if (st != TGP_OK) return st;
    if (made) {
        st = !ctx->plan_upload ? TGP_OK : (!P.blob ? plan_upload(ctx, d, P) : put_flat(ctx, P));
        ctx->times.plan_ms = now_ms() - t0;
        return st;
    }
    const int D = ctx_stack_slots(ctx);
    if (!split) d->other.reserve = nullptr;  // a flat plan with a block of its own
    const size_t budget = plan_budget(ctx, d);
    PlanJob w(d, cases, D, rows_in(budget, cases));
    w.budget = budget;
    set_split(w, dom, split);
    w.pl.team = &ctx->team;
    ScratchLoan loan(ctx, w.pl);
    w.code.swap(ctx->spare_code);
    w.code.clear();
    plan_prepare(w, ctx->fold != 0, kPlanThreads);
    const double tf0 = now_ms();
    st = fold_run(ctx, {&w});
    if (st != TGP_OK) return st;
    ctx->times.plan_fold_ms = now_ms() - tf0;
    st = plan_decide_emit_fill(w, D, ctx->reorder != 0, ctx->cache_access_cost, ctx->fold, kPlanThreads);
    if (st != TGP_OK && w.pl.tables_over && d->other.cases >= 0) {
        keep_flat(d);
        st = !ctx->plan_upload ? TGP_OK : (!P.blob ? plan_upload(ctx, d, P) : put_flat(ctx, P));
        ctx->times.plan_ms = now_ms() - t0;
        return st;
    }
    if (st != TGP_OK) return fail(ctx, st, "%s", w.err.c_str());
    if (ctx->plan_upload) {
        // the fill goes to the device (and, through after_fill, to work)
        // while the root programs are emitted
        st = plan_upload_fill(ctx, P);
        if (st == TGP_OK && after_fill) st = after_fill();
        if (st != TGP_OK) return st;
    }
    plan_emit_roots(w, kPlanThreads);
    ctx->times.plan_decide_ms = w.t_decide;
    ctx->times.plan_emit_ms = w.t_emit;
    if (ctx->plan_upload) {
        st = plan_upload_roots(ctx, d, P);
        if (st != TGP_OK) return st;
    }
    ctx->times.plan_ms = now_ms() - t0;
    return TGP_OK;
}

// The flat plan beside d's plan with tables, made from what that one keeps: no
// allocation, and no device work but put_flat's.  Returns it, or nullptr.
static Plan *flat_in_reserve(tgp_ctx ctx, tgp_dag d) {
    if (d->plan.split) std::swap(d->plan, d->other);
    Plan &P = d->plan, &with = d->other;
    if (!with.split || !with.reserve || P.blob) return nullptr;
    if (P.cases != with.cases) {
        const int D = ctx_stack_slots(ctx);
        PlanJob w(d, with.cases, D, rows_in(with.budget, with.cases));
        w.budget = with.budget;
        w.pl.team = &ctx->team;
        ScratchLoan loan(ctx, w.pl);
        plan_prepare(w, ctx->fold != 0, kPlanThreads);
        w.pl.fold_val = with.fold_val;
        if (plan_decide_emit(w, D, ctx->reorder != 0, ctx->cache_access_cost, ctx->fold, kPlanThreads) != TGP_OK) {
            P = Plan();
            return nullptr;
        }
    }
    if (flat_bytes(P) > with.reserve_bytes) return nullptr;
    char *b = static_cast<char *>(with.reserve);
    auto part = [&](size_t bytes) {
        char *p = b;
        b += (bytes + 255) & ~(size_t)255;
        return p;
    };
    P.blob = with.reserve;
    with.reserve = nullptr;
    // (the descriptors count from the first word of all the code)
    P.code_dev = P.code_roots_dev = reinterpret_cast<uint2 *>(part(sizeof(uint2) * P.code_host.size()));
    P.fill_dev = reinterpret_cast<ProgDesc *>(part(sizeof(ProgDesc) * P.fill_host.size()));
    P.reduce_dev = reinterpret_cast<ProgDesc *>(part(sizeof(ProgDesc) * P.reduce_host.size()));
    P.store_dev = reinterpret_cast<ProgDesc *>(part(sizeof(ProgDesc) * P.store_host.size()));
    P.ind_rows_dev = reinterpret_cast<int32_t *>(part(sizeof(int32_t) * P.ind_rows_host.size()));
    P.put = true;
    return &P;
}

tgp_status build_plans(tgp_ctx ctx, int32_t n, const tgp_dag *dags, const tgp_domain *doms) {
    const double t0 = now_ms();
    // one plan per distinct DAG, for the largest domain it is evaluated on
    // (the cache budget in rows is tightest there)
    // (split: the domain's, when every domain of the DAG has one shape: the
    // tables are planned for it)
    struct Want {
        tgp_domain dom;
        int32_t split;
    };
    std::unordered_map<tgp_dag, Want> want;
    std::vector<tgp_dag> order;
    // Jobs with tables beside flat ones are launched apart, each launch as long
    // as its longest program.  While the ones with tables have few work items,
    // all are planned flat: two lines and two squares of 200 trees to depth 8
    // take 135 us flat and 186 us apart at sides of 64 and 128, 240 and 255 us at
    // 256 (102 thousand items), 704 and 532 us at 512.
    constexpr int64_t kApartItems = 1 << 17;
    int64_t items = 0;
    bool flat_job = false;
    for (int32_t i = 0; i < n; ++i)
        if (wanted_split(ctx, dags[i], doms[i]))
            items += dags[i]->stats.n_roots * ((doms[i]->cases + kWideCols - 1) / kWideCols);
        else
            flat_job = true;
    const bool apart = !flat_job || items > kApartItems;
    for (int32_t i = 0; i < n; ++i) {
        const int32_t split = apart ? wanted_split(ctx, dags[i], doms[i]) : 0;
        auto it = want.find(dags[i]);
        if (it == want.end()) {
            want.emplace(dags[i], Want{doms[i], split});
            order.push_back(dags[i]);
        } else {
            Want &w = it->second;
            if (split != w.split || memcmp(doms[i]->shape, w.dom->shape, sizeof w.dom->shape) != 0) w.split = 0;
            if (doms[i]->cases > w.dom->cases) w.dom = doms[i];
        }
    }
    const int D = ctx_stack_slots(ctx);
    std::vector<std::unique_ptr<PlanJob>> jobs;
    for (tgp_dag d : order) {
        const Want &wd = want[d];
        const int64_t c = wd.dom->cases;
        int32_t split = 0;
        bool made = false;
        const tgp_status cs = choose_plan(ctx, d, wd.dom, wd.split, &made, &split);
        if (cs != TGP_OK) return cs;
        if (made) continue;
        const size_t budget = plan_budget(ctx, d);
        jobs.emplace_back(new PlanJob(d, c, D, rows_in(budget, c)));
        jobs.back()->budget = budget;
        set_split(*jobs.back(), wd.dom, split);
    }
    if (jobs.empty()) {
        ctx->times.plan_ms = now_ms() - t0;
        return TGP_OK;
    }
    // largest first, taken by host threads in turn
    std::stable_sort(jobs.begin(), jobs.end(), [](const std::unique_ptr<PlanJob> &a, const std::unique_ptr<PlanJob> &b) {
        return a->d->stats.dag_nodes > b->d->stats.dag_nodes;
    });
    const unsigned hw = usable_cpus();
    const int T = team_size(&ctx->team, (int)std::min<size_t>(std::min<unsigned>(16, hw), jobs.size()));
    auto parallel = [&](auto &&fn) {
        std::atomic<size_t> next{0};
        auto run = [&]() {
            for (size_t i; (i = next.fetch_add(1)) < jobs.size();) fn(*jobs[i]);
        };
        run_threads(&ctx->team, T, [&](int) { run(); });
    };
    const bool fold = ctx->fold != 0;
    parallel([&](PlanJob &w) { plan_prepare(w, fold); });
    const double tf0 = now_ms();
    std::vector<PlanJob *> ptrs;
    for (auto &w : jobs) ptrs.push_back(w.get());
    tgp_status st = fold_run(ctx, ptrs);
    if (st != TGP_OK) return st;
    const double tf1 = now_ms();
    const bool reorder = ctx->reorder != 0;
    const double access = ctx->cache_access_cost;
    const int fold_flag = ctx->fold;
    const int emit_threads = T > 1 ? 1 : 8;
    if (T == 1)
        for (auto &w : jobs) w->pl.team = &ctx->team;
    parallel([&](PlanJob &w) {
        w.st = plan_decide_emit(w, D, reorder, access, fold_flag, emit_threads);
        if (w.st != TGP_OK && w.pl.tables_over && w.d->other.cases >= 0) {
            keep_flat(w.d);
            w.st = TGP_OK;
        }
        if (w.st != TGP_OK) w.d->plan.cases = -1;
    });
    for (auto &w : jobs)
        if (w->st != TGP_OK) return fail(ctx, w->st, "%s", w->err.c_str());
    const double tf2 = now_ms();
    ctx->times.plan_fold_ms = tf1 - tf0;
    ctx->times.plan_decide_ms = tf2 - tf1;
    ctx->times.plan_emit_ms = 0;
    ctx->times.plan_ms = tf2 - t0;
    return TGP_OK;
}

// Work split: each work item is one program over tiles_per_stripe tiles of
// 64*K cases.  Items are kept short (at most 16 tiles) so that a launch of
// programs of very different lengths balances over 256 CUs, but long enough
// that the per-item setup (program descriptor, partial-sum write) stays small.
void choose_split(tgp_ctx ctx, int64_t n_progs, int64_t cases, int K, int32_t *stripes,
                         int32_t *tiles_per) {
    const int64_t tile = 64 * (int64_t)K;
    const int64_t n_tiles = (cases + tile - 1) / tile;
    int64_t tps;
    if (ctx->force_tiles > 0) {
        tps = ctx->force_tiles;
    } else {
        const int64_t target_items = 1 << 19;
        const int64_t total = n_tiles * std::max<int64_t>(n_progs, 1);
        const int64_t cap = ctx->tile_cap > 0 ? ctx->tile_cap : 16;
        tps = std::max<int64_t>(1, std::min<int64_t>(cap, total / target_items));
    }
    tps = std::max<int64_t>(1, std::min(tps, n_tiles));
    *tiles_per = (int32_t)tps;
    *stripes = (int32_t)((n_tiles + tps - 1) / tps);
}

int choose_K(tgp_ctx ctx, int64_t cases, const Plan &P) {
    if (P.split) return kTableK;
    if (ctx->stack_lds) return 2;  // the LDS-stack interpreter
    if (P.ext) return 4;  // the register-stack interpreter built with the bitwise operators and warp
    if (ctx->force_K) return ctx->force_K;
    return cases >= 64 * 4 * 4 ? 4 : 2;
}

void fill_job(JobDesc &j, tgp_domain dom, const uint2 *code, const float *cache) {
    memset(&j, 0, sizeof j);
    j.code = code;
    j.n_cases = (int32_t)dom->cases;
    j.ndim = dom->ndim;
    for (int k = 0; k < 3; ++k) {
        j.shape[k] = (int32_t)dom->shape[k];
        j.stride[k] = (int32_t)dom->stride[k];
        j.coord[k] = dom->coord[k] ? dom->coord[k] : dom->coord[0];
    }
    for (int k = 0; k < 2; ++k) div_magic((uint32_t)dom->stride[k], &j.div_m[k], &j.div_s[k]);
    j.cache = cache;
    j.case_base = 0;
    j.cache_stride = j.out_stride = j.target_stride = dom->cases;
    for (int k = 0; k < 2; ++k) {
        j.warp_lo[k] = (float)dom->lo[k];
        j.warp_scale[k] = dom->shape[k] > 1 ? (float)((double)(dom->shape[k] - 1) / (dom->hi[k] - dom->lo[k])) : 0.0f;
    }
}

void fill_table_fields(JobDesc &j, const Plan &P, tgp_domain dom, float *tables) {
    if (!P.split) return;
    j.row_tab = tables;
    j.col_tab = tables + P.row_bytes(*dom) / sizeof(float);
    j.row_bytes = (uint32_t)row_table_stride(*dom, P.split);
    j.col_bytes = (uint32_t)col_table_stride(*dom, P.split);
    j.n_cols = (uint32_t)dom->cols(P.split);
    div_magic(j.n_cols, &j.col_m, &j.col_s);
}

void fill_table_job(JobDesc &j, const Plan &P, tgp_domain dom, const uint2 *code, float *tables, int which) {
    memset(&j, 0, sizeof j);
    j.code = code;
    // the axes of this side of the split (none: one entry that no program uses)
    const int k0 = which ? std::min<int>(P.split, dom->ndim) : 0;
    const int k1 = which ? dom->ndim : std::min<int>(P.split, dom->ndim);
    int64_t st = 1;
    j.ndim = std::max(1, k1 - k0);
    for (int k = 0; k < 3; ++k) {
        j.shape[k] = j.stride[k] = 1;
        j.coord[k] = dom->coord[0];
    }
    for (int k = k1 - 1; k >= k0; --k) {
        j.shape[k - k0] = (int32_t)dom->shape[k];
        j.stride[k - k0] = (int32_t)st;
        j.coord[k - k0] = dom->coord[k];
        st *= dom->shape[k];
    }
    j.n_cases = (int32_t)st;
    for (int k = 0; k < 2; ++k) div_magic((uint32_t)j.stride[k], &j.div_m[k], &j.div_s[k]);
    float *tab = which ? tables + P.row_bytes(*dom) / sizeof(float) : tables;
    j.cache = tab;  // lower levels' entries
    j.out = tab;
    j.cache_stride = j.out_stride =
        (int64_t)((which ? col_table_stride(*dom, P.split) : row_table_stride(*dom, P.split)) / sizeof(float));
}

static void fill_args(InterpArgs &a, tgp_domain dom, const uint2 *code, const float *cache) {
    memset(&a, 0, sizeof a);
    fill_job(a.job, dom, code, cache);
}

// The cache-fill launches of d's plan, writing its cache rows to `cache`.
static tgp_status fill_into(tgp_ctx ctx, tgp_dag d, tgp_domain dom, int K, float *cache, float *tables) {
    const Plan &P = d->plan;
    record(ctx, 0);
    ctx->fill_recorded = ctx->timing;
    for (size_t l = 0; l < (size_t)P.levels(); ++l) {
        if (l < P.tab_level.size()) {
            const Plan::TabLevel &t = P.tab_level[l];
            TableArgs ta;
            int64_t entries = 0;
            for (int which = 0; which < 2; ++which) {
                JobDesc &j = ta.job[which];
                fill_table_job(j, P, dom, P.code_dev, tables, which);
                ta.n_progs[which] = which ? t.last - t.mid : t.mid - t.first;
                entries = std::max<int64_t>(entries, j.n_cases);
            }
            const int tk = entries >= 64 * 4 ? 4 : 2;
            for (int which = 0; which < 2; ++which) {
                JobDesc &j = ta.job[which];
                choose_split(ctx, ta.n_progs[which], j.n_cases, tk, &j.n_stripes, &j.tiles_per_stripe);
            }
            ta.progs = P.tab_dev + t.first;
            HCHK(ctx, launch_tables(tk, ta, ctx->stream));
        }
        if (l + 1 >= P.level_first.size()) continue;
        const int32_t b = P.level_first[l], e = P.level_first[l + 1];
        if (e == b) continue;
        InterpArgs a;
        fill_args(a, dom, P.code_dev, cache);
        fill_table_fields(a.job, P, dom, tables);
        a.progs = P.fill_dev + b;
        a.n_progs = e - b;
        choose_split(ctx, a.n_progs, dom->cases, K, &a.job.n_stripes, &a.job.tiles_per_stripe);
        a.job.out = cache;
        HCHK(ctx, launch_interp(K, P.D, true, a, ctx->stream, form_of(P, *dom)));
    }
    record(ctx, 1);
    return TGP_OK;
}

static tgp_status run_fill(tgp_ctx ctx, tgp_dag d, tgp_domain dom, int K, float **cache_out) {
    const Plan &P = d->plan;
    *cache_out = nullptr;
    ctx->fill_recorded = false;
    if (P.n_slots == 0 && P.tab_host.empty()) return TGP_OK;
    const size_t bytes = sizeof(float) * (size_t)P.n_slots * (size_t)dom->cases;
    if (P.n_slots) HCHK(ctx, ensure(ctx->cache, bytes));
    // Like the cache rows, the tables hold one evaluation's values at a time.
    // (tgp_fitness_noalloc has tables of its own: a captured call may be
    // replayed beside this one on another stream.)  Their size differs from one
    // generation to the next: they grow to powers of two.
    size_t tab = 256;
    while (tab < P.tables_bytes(*dom)) tab <<= 1;
    if (P.split) HCHK(ctx, ensure(ctx->tables, tab));
    float *cache = P.n_slots ? (float *)ctx->cache.p : nullptr;
    *cache_out = cache;
    return fill_into(ctx, d, dom, K, cache, (float *)ctx->tables.p);
}

// The plan of d for dom with its cache filled (fill launches queued on the
// context's stream).  A new plan's fill is queued as soon as its programs
// are on the device, while the host still emits the root programs; the
// fill's operand stack form follows the fill programs alone (they may not
// need the bitwise operators or warp when the root programs do).
static tgp_status plan_and_fill(tgp_ctx ctx, tgp_dag d, tgp_domain dom, float **cache) {
    bool filled = false;
    tgp_status st = build_plan(ctx, d, dom, [&]() {
        filled = true;
        return run_fill(ctx, d, dom, choose_K(ctx, dom->cases, d->plan), cache);
    });
    if (st != TGP_OK || filled) return st;
    return run_fill(ctx, d, dom, choose_K(ctx, dom->cases, d->plan), cache);
}

tgp_status check_eval_args(tgp_ctx ctx, tgp_dag d, tgp_domain dom) {
    if (!ctx || !d || !dom) return fail(ctx, TGP_EINVAL, "NULL argument");
    if (d->ctx != ctx || dom->ctx != ctx) return fail(ctx, TGP_EINVAL, "handles of another context");
    if (d->stats.max_var >= dom->ndim)
        return fail(ctx, TGP_ESHAPE, "a tree uses axis %lld but the domain has %d axes",
                    (long long)d->stats.max_var, dom->ndim);
    return TGP_OK;
}

static void record_work(tgp_ctx ctx, tgp_dag d, tgp_domain dom, bool fitness) {
    const Plan &P = d->plan;
    tgp_work_stats &w = ctx->work;
    const double cases = (double)dom->cases;
    w.credited_node_evals = d->stats.dag_nodes * dom->cases;
    const double rows = P.split ? (double)dom->rows(P.split) : 0, cols = P.split ? (double)dom->cols(P.split) : 0;
    const int64_t tab_cells = (int64_t)(P.n_tab[0] * rows + P.n_tab[1] * cols);
    w.executed_node_evals = (int64_t)(P.exec_per_case * cases + P.exec_tab[0] * rows + P.exec_tab[1] * cols);
    w.cached_nodes = P.n_slots + P.n_tab[0] + P.n_tab[1];
    w.stack_spills = P.n_spills;
    w.cache_levels = P.levels();
    w.programs = fitness ? P.n_reduce : P.n_store;
    w.instructions = P.instructions;
    w.algorithmic_valu = P.valu_dag_per_case * cases;
    w.executed_valu_fill = P.valu_fill_per_case * cases;
    w.executed_valu_roots = P.valu_roots_per_case * cases;
    w.cache_bytes_written = ((int64_t)P.n_slots * dom->cases + tab_cells) * 4;
    w.cache_bytes_read = P.cache_reads_per_case * dom->cases * 4;
    w.folded_nodes = P.n_folded;
}

extern "C" {

// Whether p is host memory (pageable or pinned) rather than device-resident.
static bool is_host_memory(const void *p) {
    hipPointerAttribute_t attr{};
    if (hipPointerGetAttributes(&attr, p) != hipSuccess) {
        (void)hipGetLastError();  // an unknown (pageable) pointer: clear the error it leaves
        return true;
    }
    return attr.type == hipMemoryTypeHost || attr.type == hipMemoryTypeUnregistered;
}

tgp_status tgp_fitness(tgp_ctx ctx, tgp_dag d, tgp_domain dom, const float *target_dev, int32_t loss,
                       double *out) {
    tgp_status st = check_eval_args(ctx, d, dom);
    if (st != TGP_OK) return st;
    if (loss != TGP_RMSE && loss != TGP_MSE) return fail(ctx, TGP_EINVAL, "loss must be TGP_RMSE or TGP_MSE");
    if (d->n_ind == 0) return TGP_OK;
    if (!target_dev || !out) return fail(ctx, TGP_EINVAL, "NULL target or output");
    HCHK(ctx, hipSetDevice(ctx->device));
    const bool host_out = is_host_memory(out);
    double *out_dev = out;
    if (host_out) {
        HCHK(ctx, ensure(ctx->fit_out, sizeof(double) * (size_t)d->n_ind));
        out_dev = static_cast<double *>(ctx->fit_out.p);
    }
    float *cache = nullptr;
    st = plan_and_fill(ctx, d, dom, &cache);
    if (st != TGP_OK) return st;
    const Plan &P = d->plan;
    const int K = choose_K(ctx, dom->cases, P);
    InterpArgs a;
    fill_args(a, dom, P.code_roots_dev, cache);
    fill_table_fields(a.job, P, dom, (float *)ctx->tables.p);
    a.progs = P.reduce_dev;
    a.n_progs = P.n_reduce;
    choose_split(ctx, a.n_progs, dom->cases, K, &a.job.n_stripes, &a.job.tiles_per_stripe);
    a.job.target = target_dev;
    HCHK(ctx, ensure(ctx->partial, sizeof(float2) * (size_t)a.n_progs * (size_t)a.job.n_stripes));
    a.job.partial = (float2 *)ctx->partial.p;
    record(ctx, 2);
    HCHK(ctx, launch_interp(K, P.D, false, a, ctx->stream, form_of(P, *dom)));
    record(ctx, 3);
    record(ctx, 4);
    HCHK(ctx, launch_finalize(a.job.partial, P.ind_rows_dev, d->n_ind, d->n_ch, a.job.n_stripes,
                              (double)d->n_ch * (double)dom->cases, loss, out_dev, ctx->stream));
    record(ctx, 5);
    if (host_out) {
        HCHK(ctx, hipMemcpyAsync(out, out_dev, sizeof(double) * (size_t)d->n_ind, hipMemcpyDeviceToHost,
                                 ctx->stream));
        HCHK(ctx, hipStreamSynchronize(ctx->stream));
    }
    ctx->times.interp_items = (int64_t)a.n_progs * a.job.n_stripes;
    ctx->times.cases_per_lane = K;
    ctx->times.tiles_per_item = a.job.tiles_per_stripe;
    record_work(ctx, d, dom, true);
    return TGP_OK;
}

tgp_status tgp_fitness_noalloc(tgp_ctx ctx, tgp_dag d, tgp_domain dom, const float *target_dev,
                               int32_t loss, double *out_dev) {
    tgp_status st = check_eval_args(ctx, d, dom);
    if (st != TGP_OK) return st;
    if (loss != TGP_RMSE && loss != TGP_MSE) return fail(ctx, TGP_EINVAL, "loss must be TGP_RMSE or TGP_MSE");
    if (d->n_ind == 0) return TGP_OK;
    if (!target_dev || !out_dev) return fail(ctx, TGP_EINVAL, "NULL target or output");
    if (is_host_memory(out_dev) || is_host_memory(target_dev))
        return fail(ctx, TGP_EINVAL, "tgp_fitness_noalloc takes device-resident target and output");
    HCHK(ctx, hipSetDevice(ctx->device));
    if (ctx->device >= kMaxDevices || !g_scratch_ptr[ctx->device])
        return fail(ctx, TGP_EHIP, "no scratch address for device %d: %s", ctx->device,
                    ctx->device < kMaxDevices ? hipGetErrorString(g_scratch_err[ctx->device]) : "device index");
    // What a call with plan Q puts into the scratch: the partial sums, the cache
    // rows and the tables (unless the plan keeps a block for them).
    struct Layout {
        int32_t stripes, tiles;
        size_t partial, rows, tables, total;
        float *own;
    };
    auto layout = [&](const Plan &Q) {
        auto up = [](size_t n) { return (n + 255) & ~(size_t)255; };
        Layout l;
        choose_split(ctx, Q.n_reduce, dom->cases, choose_K(ctx, dom->cases, Q), &l.stripes, &l.tiles);
        l.partial = up(sizeof(float2) * (size_t)Q.n_reduce * (size_t)l.stripes);
        l.rows = sizeof(float) * (size_t)Q.n_slots * (size_t)dom->cases;
        l.own = Q.planned_shape(*dom) ? static_cast<float *>(Q.noalloc_tables) : nullptr;
        l.tables = l.own ? 0 : Q.tables_bytes(*dom);
        l.total = l.tables ? up(l.partial + l.rows) + l.tables : l.partial + l.rows;
        return l;
    };
    // The best plan for dom's shape if it is on the device and fits; else any
    // that does, the flat one made for it where only one with tables is there.
    auto ready = [&](const Plan *Q) {
        return Q && plan_current(ctx, *Q, dom->cases) && Q->blob && Q->code_roots_dev;
    };
    auto fits = [&](const Plan *Q) { return ready(Q) && layout(*Q).total <= kNoAllocScratchBytes; };
    if (!ready(&d->plan) && !ready(&d->other))
        return fail(ctx, TGP_EINVAL,
                    "the DAG has no plan for a domain of %lld cases under this context's settings "
                    "(evaluate it once with tgp_fitness or tgp_evaluate)", (long long)dom->cases);
    const int32_t want = wanted_split(ctx, d, dom);
    auto first_fit = [&](bool with_tables) -> Plan * {
        for (Plan *Q : {&d->plan, &d->other})
            if ((Q->split > 0) == with_tables && fits(Q)) return Q;
        return nullptr;
    };
    Plan *chosen = first_fit(want > 0);
    if (!chosen && want > 0) chosen = first_fit(false);
    if (!chosen && flat_in_reserve(ctx, d)) chosen = first_fit(false);
    if (!chosen) chosen = first_fit(true);
    if (!chosen) {
        const Plan &Q = ready(&d->plan) ? d->plan : d->other;
        const Layout l = layout(Q);
        return fail(ctx, TGP_ENOMEM,
                    "needs %zu bytes of scratch (%zu of partial sums, %zu of cache rows, %zu of tables); "
                    "tgp_fitness_noalloc has %zu", l.total, l.partial, l.rows, l.tables, kNoAllocScratchBytes);
    }
    if (chosen != &d->plan) std::swap(d->plan, d->other);
    st = put_flat(ctx, d->plan);
    if (st != TGP_OK) return st;
    const Plan &P = d->plan;
    const int K = choose_K(ctx, dom->cases, P);
    const Layout l = layout(P);
    InterpArgs a;
    fill_args(a, dom, P.code_roots_dev, nullptr);
    a.progs = P.reduce_dev;
    a.n_progs = P.n_reduce;
    a.job.n_stripes = l.stripes;
    a.job.tiles_per_stripe = l.tiles;
    // Every (program, stripe) pair and every cache row is written before it
    // is read, so nothing in the scratch needs clearing between calls.
    char *base = static_cast<char *>(g_scratch_ptr[ctx->device]);
    float *cache = P.n_slots ? reinterpret_cast<float *>(base + l.partial) : nullptr;
    float *tables = l.own ? l.own : reinterpret_cast<float *>(base + l.total - l.tables);
    ctx->fill_recorded = false;
    if (P.n_slots || !P.tab_host.empty()) {
        st = fill_into(ctx, d, dom, K, cache, tables);
        if (st != TGP_OK) return st;
    }
    fill_table_fields(a.job, P, dom, tables);
    a.job.cache = cache;
    a.job.target = target_dev;
    a.job.partial = reinterpret_cast<float2 *>(base);
    record(ctx, 2);
    HCHK(ctx, launch_interp(K, P.D, false, a, ctx->stream, form_of(P, *dom)));
    record(ctx, 3);
    record(ctx, 4);
    HCHK(ctx, launch_finalize(a.job.partial, P.ind_rows_dev, d->n_ind, d->n_ch, a.job.n_stripes,
                              (double)d->n_ch * (double)dom->cases, loss, out_dev, ctx->stream));
    record(ctx, 5);
    ctx->times.interp_items = (int64_t)a.n_progs * a.job.n_stripes;
    ctx->times.cases_per_lane = K;
    ctx->times.tiles_per_item = a.job.tiles_per_stripe;
    record_work(ctx, d, dom, true);
    return TGP_OK;
}

tgp_status tgp_evaluate(tgp_ctx ctx, tgp_dag d, tgp_domain dom, float *out_dev) {
    tgp_status st = check_eval_args(ctx, d, dom);
    if (st != TGP_OK) return st;
    if (d->stats.n_roots == 0) return TGP_OK;
    if (!out_dev) return fail(ctx, TGP_EINVAL, "NULL output");
    HCHK(ctx, hipSetDevice(ctx->device));
    float *cache = nullptr;
    st = plan_and_fill(ctx, d, dom, &cache);
    if (st != TGP_OK) return st;
    const Plan &P = d->plan;
    const int K = choose_K(ctx, dom->cases, P);
    InterpArgs a;
    fill_args(a, dom, P.code_roots_dev, cache);
    fill_table_fields(a.job, P, dom, (float *)ctx->tables.p);
    a.progs = P.store_dev;
    a.n_progs = P.n_store;
    choose_split(ctx, a.n_progs, dom->cases, K, &a.job.n_stripes, &a.job.tiles_per_stripe);
    a.job.out = out_dev;
    record(ctx, 2);
    HCHK(ctx, launch_interp(K, P.D, true, a, ctx->stream, form_of(P, *dom)));
    record(ctx, 3);
    record(ctx, 4);
    record(ctx, 5);
    ctx->times.interp_items = (int64_t)a.n_progs * a.job.n_stripes;
    ctx->times.cases_per_lane = K;
    ctx->times.tiles_per_item = a.job.tiles_per_stripe;
    const size_t row = sizeof(float) * (size_t)dom->cases;
    for (int64_t r = 0; r < d->stats.n_roots; ++r)
        if (P.dup_src[r] >= 0)
            HCHK(ctx, hipMemcpyAsync((char *)out_dev + row * r, (char *)out_dev + row * P.dup_src[r], row,
                                     hipMemcpyDeviceToDevice, ctx->stream));
    record_work(ctx, d, dom, false);
    return TGP_OK;
}

tgp_status tgp_last_work(tgp_ctx ctx, tgp_work_stats *out) {
    if (!ctx || !out) return fail(ctx, TGP_EINVAL, "NULL argument");
    *out = ctx->work;
    return TGP_OK;
}

}  // extern "C"
