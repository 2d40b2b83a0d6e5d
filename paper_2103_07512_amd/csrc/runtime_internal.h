// runtime_internal.h -- host objects of libtgp shared by the translation
// units of the runtime (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <functional>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "tgp_internal.h"

using namespace tgp;

// ------------------------------------------------------------------ objects
struct DevBuf {
    void *p = nullptr;
    size_t cap = 0;
};

// Host threads that a context keeps for planning (creating them for every
// phase of every plan costs more than most phases): at most kMaxWorkers, made
// on first use and joined when the context is destroyed.  Used by the
// context's one host thread at a time.
class HostTeam {
public:
    ~HostTeam();
    // Makes the threads for rounds of T; returns how many a round can have (fewer
    // when the process gets no more threads).
    int grow(int T);
    // Runs fn(t) for t = 0 .. T-1, t = 0 on the calling thread, and returns
    // when all have returned.  T is at most what grow returned.
    void run(int T, const std::function<void(int)> &fn);

private:
    static constexpr int kMaxWorkers = 15;
    void work(int id, uint64_t seen);
    std::vector<std::thread> workers_;
    std::mutex m_;
    std::condition_variable cv_;
    std::atomic<uint64_t> round_{0};
    std::atomic<int> left_{0};
    int want_ = 0;
    const std::function<void(int)> *fn_ = nullptr;
    bool stop_ = false;
};

// Host arrays that a context keeps from one DAG and plan to the next (their
// pages would otherwise be mapped and cleared anew every generation): one
// set, of the largest DAG seen, given back with the context.
struct DagArrays {
    std::vector<int32_t> op;  // op | var << 8
    std::vector<float> value;
    std::vector<int32_t> kid;  // [U][3]
    std::vector<int32_t> roots, mult, indeg, height;
    void swap(DagArrays &o) {
        op.swap(o.op);
        value.swap(o.value);
        kid.swap(o.kid);
        roots.swap(o.roots);
        mult.swap(o.mult);
        indeg.swap(o.indeg);
        height.swap(o.height);
    }
};
struct PlanScratch;  // the planner's arrays (runtime.cpp)

struct tgp_ctx_s {
    HostTeam team;
    DagArrays spare_dag;
    std::vector<uint2> spare_code;
    std::shared_ptr<PlanScratch> plan_scratch;
    int device = 0;
    hipStream_t stream = nullptr;
    size_t cache_budget = 0;
    std::string err;
    tgp_work_stats work{};
    int force_K = 0;  // 0 = automatic
    int force_tiles = 0;
    int tile_cap = 0;  // cap on automatic tiles per item (0 = 16)
    int batch_persistent = 1;  // batched launches: persistent waves (1) or one wave per item
    tgp_batch batch = nullptr;  // kept by tgp_fitness_batch
    int reorder = 1;                     // Sethi-Ullman child order
    bool plan_upload = true;             // plans also kept on the device
    int stack_lds = 0;                   // operand stack in LDS (1) or registers (0)
    int fold = 1;                        // constant folding
    int commute = 0;                     // hash-consing up to operand order of commuting operators
    int rewrite = 0;                     // identity rewrites while hash-consing
    double cache_access_cost = 20.0;     // < 0: no benefit-driven caching
    DevBuf partial, cache;
    DevBuf fit_out;  // device copy of fitness values bound for host memory
    DevBuf tables;   // tables of one evaluation, filled by it
    DevicePool pool;             // DAG, plan and population blocks
    void *pin = nullptr;         // pinned staging for uploads and readbacks
    size_t pin_cap = 0;
    hipEvent_t pin_ev = nullptr; // recorded after the last copy out of `pin`
    bool pin_pending = false;
    bool timing = false;
    bool ev_ready = false;
    // fill begin/end, interp begin/end, finalize begin/end, then breeding:
    // shape begin, shape end = decisions begin, decisions end, copy begin/end
    hipEvent_t ev[11] = {};
    uint32_t recorded = 0;  // bit i: ev[i] has been recorded
    bool fill_recorded = false;
    tgp_timing times{};
};

inline double now_ms() {
    return std::chrono::duration<double, std::milli>(
               std::chrono::steady_clock::now().time_since_epoch())
        .count();
}

inline void record(tgp_ctx ctx, int i) {
    if (ctx->timing && ctx->ev_ready && hipEventRecord(ctx->ev[i], ctx->stream) == hipSuccess)
        ctx->recorded |= 1u << i;
}

struct tgp_domain_s {
    tgp_ctx ctx = nullptr;
    int32_t ndim = 0;
    int64_t shape[3] = {1, 1, 1};
    int64_t stride[3] = {1, 1, 1};
    int64_t cases = 0;
    double lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
    float *coord[3] = {nullptr, nullptr, nullptr};
    // The split of the axes for table programs (0: the domain is evaluated
    // flat): axes below it number the grid rows, the others the columns.
    int32_t split = 0;
    // Entries of the tables of a program split at axis s.  Any s of 1..2 has
    // a meaning on any domain (without axes on one side it has one entry).
    int64_t rows(int s) const {
        int64_t n = 1;
        for (int k = 0; k < s && k < ndim; ++k) n *= shape[k];
        return n;
    }
    int64_t cols(int s) const { return cases / rows(s); }
};

// Byte strides of the tables' subtrees on a domain split at axis s.
inline size_t table_stride(int64_t entries) { return sizeof(float) * (size_t)((entries + 15) / 16 * 16); }
inline size_t row_table_stride(const tgp_domain_s &d, int s) { return table_stride(d.rows(s)); }
inline size_t col_table_stride(const tgp_domain_s &d, int s) { return table_stride(d.cols(s)); }

// A compiled evaluation plan of one DAG for one case count.
struct Plan {
    int64_t cases = -1;
    int D = 0;                          // stack slots the programs were planned for
    bool reorder = true;
    double access_cost = 0;
    int fold = -1;
    int64_t n_folded = 0;               // constant subtrees folded
    // Table programs (split > 0): subtrees of the leading axes alone live in the
    // row table, of the trailing axes alone in the column table, the cache
    // slots hold the others.  asked: the split the plan was made for (a plan
    // whose tables did not fit falls back to flat programs, split = 0, and
    // keeps their entries in refused).  tab_rows: the grid rows of the domain
    // that the tables were admitted for; their size follows the shape, so on
    // another shape of the same size they are checked again (best_plan).
    int32_t split = 0, asked = 0;
    int64_t tab_rows = 0;
    int64_t refused[2] = {0, 0};
    size_t budget = 0;                  // the cache budget that the plan was made for
    // Beside tables: what the flat plan is made from where nothing may be
    // allocated (flat_in_reserve): the folded constants, and the end of blob_roots,
    // which then holds its programs (the two plans are given up together).
    std::vector<float> fold_val;
    void *reserve = nullptr;
    size_t reserve_bytes = 0;
    // Tables on that shape for tgp_fitness_noalloc, where its own memory cannot
    // hold them beside the rest (else null).  Nothing else uses the block.
    void *noalloc_tables = nullptr;
    bool put = false;                   // the blob is still to be written (put_flat)
    int32_t n_tab[2] = {0, 0};          // subtrees in the row and column tables
    struct TabLevel {
        int32_t first, mid, last;       // row programs [first, mid), column programs [mid, last)
    };
    std::vector<TabLevel> tab_level;    // table programs of each level
    std::vector<ProgDesc> tab_host;
    ProgDesc *tab_dev = nullptr;
    int64_t tab_code_end = 0;           // the table programs' code comes first in code_host
    double exec_tab[2] = {0, 0};        // instructions run per table entry
    int levels() const { return (int)std::max(level_first.empty() ? 0 : level_first.size() - 1, tab_level.size()); }
    size_t tables_bytes(const tgp_domain_s &d) const {
        if (!split) return 0;
        return row_bytes(d) + (size_t)n_tab[1] * col_table_stride(d, split);
    }
    // Of the shape that the tables were admitted for.
    bool planned_shape(const tgp_domain_s &d) const { return split > 0 && d.rows(split) == tab_rows; }
    size_t planned_tables_bytes() const {
        const size_t rows = (size_t)n_tab[0] * table_stride(tab_rows);
        return ((rows + 255) & ~(size_t)255) + (size_t)n_tab[1] * table_stride(cases / tab_rows);
    }
    size_t row_bytes(const tgp_domain_s &d) const {
        return ((size_t)n_tab[0] * row_table_stride(d, split) + 255) & ~(size_t)255;
    }
    int32_t n_slots = 0;
    int64_t n_spills = 0;               // cached only to bound the register stack
    std::vector<int32_t> level_first;   // fill programs of level l: [level_first[l], level_first[l+1])
    int32_t n_fill = 0;
    int32_t n_reduce = 0;               // programs for (root, channel)
    int32_t n_store = 0;                // programs for distinct roots
    std::vector<int32_t> store_rows;    // for each root r: the store program's dest row, or -1
    std::vector<int32_t> dup_src;       // for each root r: row r copies row dup_src[r] (-1: none)
    // Device copies in two pool blocks, so that the fill can start before the
    // root programs are emitted: blob holds the fill programs' code and
    // descriptors, blob_roots the root programs' code (code_roots_dev), the
    // reduce and store descriptors (code offsets relative to code_roots_dev)
    // and the individual rows.
    void *blob = nullptr, *blob_roots = nullptr;
    uint2 *code_dev = nullptr, *code_roots_dev = nullptr;
    ProgDesc *fill_dev = nullptr, *reduce_dev = nullptr, *store_dev = nullptr;
    int32_t *ind_rows_dev = nullptr;
    int64_t root_code_at = 0;           // first root instruction in code_host
    // host copies (the batched path packs them into its own buffers); code
    // offsets in all three descriptor lists are into code_host
    std::vector<uint2> code_host;
    std::vector<ProgDesc> fill_host, reduce_host, store_host;
    std::vector<int32_t> ind_rows_host;
    std::vector<int32_t> slot_node;     // DAG node held by each cache slot
    std::vector<uint8_t> slot_pre;      // slot already resident (no fill program)
    bool ext = false;                   // uses the bitwise operators, warp or the third axis
    bool warp = false;                  // uses warp
    int64_t instructions = 0;
    double exec_per_case = 0;           // instructions run per case, fitness form
    double valu_dag_per_case = 0;       // cost-model slots of each DAG node once
    double valu_fill_per_case = 0;      // cost-model slots run by the fill programs
    double valu_roots_per_case = 0;     // cost-model slots run by the reduce programs
    int64_t cache_reads_per_case = 0;   // I_CACHE instructions executed, fitness form
    // The caller guarantees that no queued kernel still reads the block.
    void release(DevicePool &pool) {
        pool.release(blob);
        pool.release(blob_roots);
        pool.release(noalloc_tables);
        blob = blob_roots = reserve = noalloc_tables = nullptr;
        put = false;
        tab_dev = nullptr;
        code_dev = code_roots_dev = nullptr;
        fill_dev = reduce_dev = store_dev = nullptr;
        ind_rows_dev = nullptr;
        cases = -1;
    }
};

struct tgp_dag_s : DagArrays {  // host copies
    tgp_ctx ctx = nullptr;
    int32_t n_ind = 0, n_ch = 0;
    tgp_dag_stats stats{};
    DagDevice dev;
    bool image_ops = false;          // a bitwise operator or warp occurs
    std::vector<uint8_t> precached;  // nodes whose values are resident (empty: none)
    bool no_tables = false;          // plans are flat on every domain
    // The plan in use.  other: the flat plan where that one has tables, or the
    // one with tables where it is flat; both are for one number of cases and
    // one set of the context's settings, and either stays as it is (a captured
    // call may read it) until a plan for others is made.
    Plan plan, other;
};

namespace tgp {
// Builds the DAG of R trees given device tokens and offsets under the
// context's hashing settings (T < 0: the token count is offsets[R], read from
// the device and checked).  The device arrays come from the context's pool
// (given back with dag_device_free once the stream has passed every use);
// *host is a copy of them in the context's pinned staging.  Blocks.
DagBuildResult build_dag_device(tgp_ctx ctx, const tgp_token *tok_dev, const int64_t *off_dev, int64_t R, int64_t T,
                                DagDevice *dev, const int32_t **host, char *err, size_t errlen);
}  // namespace tgp

// ------------------------------------------------------------------ errors
tgp_status fail(tgp_ctx ctx, tgp_status st, const char *fmt, ...);

#define HCHK(ctx, x)                                                                           \
    do {                                                                                       \
        hipError_t _e = (x);                                                                   \
        if (_e != hipSuccess)                                                                  \
            return fail(ctx, TGP_EHIP, "%s failed: %s", #x, hipGetErrorString(_e));            \
    } while (0)

inline hipError_t ensure(DevBuf &b, size_t bytes) {
    if (b.cap >= bytes && b.p) return hipSuccess;
    if (b.p) {
        hipError_t e = hipFree(b.p);
        if (e != hipSuccess) return e;
        b.p = nullptr;
        b.cap = 0;
    }
    size_t want = std::max<size_t>(bytes, 256);
    hipError_t e = hipMalloc(&b.p, want);
    if (e == hipSuccess) b.cap = want;
    return e;
}


// Pinned staging of at least `bytes`, free to be overwritten (waits for the
// copy that last read it).
hipError_t ctx_pinned(tgp_ctx ctx, size_t bytes, void **out);
// Marks the staging as read by copies enqueued on the context stream.
hipError_t ctx_pinned_enqueued(tgp_ctx ctx);

// One job of a batched step: a plan's programs over the cases
// [case_base, case_base + n_cases) of a domain.
struct StepJob {
    const Plan *plan;             // host copies of the programs are used
    tgp_domain domain;
    int32_t n_ind = 0, n_ch = 0;
    int32_t case_base = 0, n_cases = 0;
    const float *target = nullptr;   // [n_ch][domain cases]
    // Cache rows: with cache == nullptr the step allocates [slots][domain
    // cases] rows itself (slot s is row s); otherwise the plan's slot numbers
    // are rows of `cache` with stride cache_stride.
    const float *cache = nullptr;
    int64_t cache_stride = 0;
    double *acc = nullptr;        // slab running sums (nullptr: whole domain)
    int32_t first = 1, last = 1;  // first / last slab of the domain
    double *out = nullptr;        // device, [n_ind]
    int32_t loss = TGP_RMSE;
    int32_t tiles_per_item = 0;   // 0: chosen from the whole step's work
    // Programs and individual rows already on the device (nullptr: the step
    // uploads the plan's host copies).
    const uint2 *code_dev = nullptr;
    const int32_t *rows_dev = nullptr;
    // Table programs: the request's tables (nullptr: the step allocates them) and
    // whether this step fills them.
    float *tables = nullptr;
    bool fill_tables = true;
};
tgp_status batch_step(tgp_batch b, int32_t n_jobs, const StepJob *jobs, int64_t credited);

// --------------------------------------------------------------- shared helpers
extern const double kOpCost[TGP_NUM_OPS];
// Plans d for domains like dom (a no-op when its plan is current) and
// uploads the programs when the context keeps plans on the device.  When a
// new plan is uploaded, after_fill (if given) is called once the fill
// programs are on the device and before the root programs are emitted, so
// that the caller can queue the cache fill while the host emits the rest.
tgp_status build_plan(tgp_ctx ctx, tgp_dag d, tgp_domain dom,
                      const std::function<tgp_status()> &after_fill = nullptr);
// Gives up d's plans (no queued kernel reads them).
void forget_plans(tgp_ctx ctx, tgp_dag d);
// Plans many DAGs at once (host threads, one device round trip for constant
// folding); programs stay on the host.  A DAG listed more than once is
// planned once, for its largest domain.
tgp_status build_plans(tgp_ctx ctx, int32_t n, const tgp_dag *dags, const tgp_domain *doms);
// Cases per lane of a plan's launches over `cases` cases, and their form.
int choose_K(tgp_ctx ctx, int64_t cases, const Plan &P);
inline int form_of(const Plan &P, const tgp_domain_s &d) {
    if (P.split) return d.cols(P.split) % kWideCols == 0 ? kWide : kRagged;
    return P.ext ? kExt : kFlat;
}
int ctx_stack_slots(tgp_ctx ctx);
void choose_split(tgp_ctx ctx, int64_t n_progs, int64_t cases, int K, int32_t *stripes,
                  int32_t *tiles_per);
void fill_job(JobDesc &j, tgp_domain dom, const uint2 *code, const float *cache);
// The table fields of j for P's split, the tables at `tables`.
void fill_table_fields(JobDesc &j, const Plan &P, tgp_domain dom, float *tables);
// The flat job that fills the row (which = 0) or column (1) table of P.
void fill_table_job(JobDesc &j, const Plan &P, tgp_domain dom, const uint2 *code, float *tables, int which);
tgp_status check_eval_args(tgp_ctx ctx, tgp_dag d, tgp_domain dom);
