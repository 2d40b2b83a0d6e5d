// Host check of which plan a DAG is evaluated with (runtime.cpp, compiled for
// the CPU as in planner_check.cpp; no device call).  A plan's tables are
// admitted for one shape of grid; on another of the same number of cases:
//   - the plan with tables is used only where the tables are within half the
//     cache budget and a 32-bit byte offset of each, else a flat one;
//   - a DAG evaluated on several shapes in turn is planned twice at most, and
//     the plan that is not in use stays where it is;
//   - the flat plan that tgp_fitness_noalloc makes beside one with tables is the
//     one that planning flat gives, and fits the block kept for it.
#define main planner_check_main
#include "planner_check.cpp"
#undef main

namespace {

tgp_domain_s domain(tgp_ctx ctx, std::vector<int64_t> shape) {
    tgp_domain_s s;
    s.ctx = ctx;
    s.ndim = (int32_t)shape.size();
    s.cases = 1;
    for (size_t k = 0; k < shape.size(); ++k) s.cases *= s.shape[k] = shape[k];
    s.split = domain_split(s);
    return s;
}

// n trees x + y * c, each with a constant of its own: n column entries, one row entry.
void column_trees(tgp_dag_s &d, tgp_ctx ctx, int n) {
    Builder b(d);
    d.ctx = ctx;
    d.n_ind = n;
    d.n_ch = 1;
    for (int i = 0; i < n; ++i)
        d.roots.push_back(b.add_tree({{TGP_VAR, 0, 0}, {TGP_VAR, 1, 0}, {TGP_CONST, 0, (float)(i + 1)}, {TGP_MULT, 0, 0},
                                      {TGP_ADD, 0, 0}}));
    d.stats.dag_nodes = (int64_t)d.op.size();
    d.stats.n_roots = n;
}

int g_planned = 0;

// What build_plan does on the host.
void use(tgp_ctx ctx, tgp_dag_s &d, tgp_domain_s dom) {
    bool made = false;
    int32_t split = 0;
    CHECK(choose_plan(ctx, &d, &dom, wanted_split(ctx, &d, &dom), &made, &split) == TGP_OK, "choose_plan failed\n");
    if (!made) {
        ++g_planned;
        const size_t budget = plan_budget(ctx, &d);
        PlanJob w(&d, dom.cases, 8, rows_in(budget, dom.cases));
        w.budget = budget;
        set_split(w, &dom, split);
        plan_prepare(w, true);
        const tgp_status st = plan_decide_emit(w, 8, true, ctx->cache_access_cost, 1, 1);
        if (st != TGP_OK && w.pl.tables_over && d.other.cases >= 0) keep_flat(&d);
        else CHECK(st == TGP_OK, "plan: status %d\n", st);
    }
    const Plan &P = d.plan;
    CHECK(P.cases == dom.cases, "the plan in use is for %lld cases\n", (long long)P.cases);
    if (!P.split) return;
    const double row = (double)P.n_tab[0] * row_table_stride(dom, P.split);
    const double col = (double)P.n_tab[1] * col_table_stride(dom, P.split);
    CHECK(row < 4294967296.0 && col < 4294967296.0, "%lld x %lld: tables of %.0f and %.0f bytes\n",
          (long long)dom.rows(P.split), (long long)dom.cols(P.split), row, col);
    CHECK(row + col <= ctx->cache_budget / 2.0, "tables of %.0f bytes, budget %zu\n", row + col, ctx->cache_budget);
}

// The folded subtrees' values (no variable: any case).
void fold(tgp_dag_s &d, PlanJob &w) {
    if (w.pl.folded.empty()) return;
    const int64_t U = d.stats.dag_nodes;
    w.pl.fold_val.assign(U, 0.0f);
    for (int64_t n = 0; n < U; ++n) {
        const int op = d.op[n] & 0xff;
        const int32_t *k = &d.kid[3 * n];
        float *v = w.pl.fold_val.data();
        v[n] = kArity[op] == 0 ? d.value[n] : apply(op, v[k[0]], k[1] >= 0 ? v[k[1]] : 0, k[2] >= 0 ? v[k[2]] : 0);
    }
}

template <class T>
bool same(const std::vector<T> &a, const std::vector<T> &b) {
    return a.size() == b.size() && memcmp(a.data(), b.data(), sizeof(T) * a.size()) == 0;
}

void check_reserve(tgp_ctx ctx, Gen &g, int n_ind, int n_ch, int d_max, tgp_domain_s dom) {
    tgp_dag_s d;
    d.ctx = ctx;
    make_dag(d, g, n_ind, n_ch, d_max);
    std::vector<int64_t> size(d.op.size(), 1);
    for (size_t n = 0; n < d.op.size(); ++n)
        for (int j = 0; j < 3; ++j)
            if (d.kid[3 * n + j] >= 0) size[n] += size[d.kid[3 * n + j]];
    for (int32_t r : d.roots) d.stats.tree_nodes += size[r];
    for (int32_t o : d.op) d.stats.dag_internal += kArity[o & 0xff] > 0;
    Plan flat;
    for (int32_t split : {0, dom.split}) {
        d.plan = Plan();
        PlanJob w(&d, dom.cases, 8, rows_in(ctx->cache_budget, dom.cases));
        w.budget = ctx->cache_budget;
        set_split(w, &dom, split);
        plan_prepare(w, true);
        fold(d, w);
        const tgp_status st = plan_decide_emit(w, 8, true, ctx->cache_access_cost, 1, 1);
        CHECK(st == TGP_OK && d.plan.split == split, "U=%lld: status %d\n", (long long)d.stats.dag_nodes, st);
        if (!split) flat = d.plan;
    }
    const size_t bound = flat_bytes_bound(d, dom.cases), need = flat_bytes(flat);
    const bool fits = sizeof(float) * (size_t)flat.n_slots * (size_t)dom.cases <= kNoAllocScratchBytes;
    CHECK(!fits || need <= bound, "U=%lld: %zu bytes of flat programs, bound %zu\n", (long long)d.stats.dag_nodes, need, bound);
    std::vector<char> block(bound);
    d.plan.reserve = block.data();
    d.plan.reserve_bytes = bound;
    const size_t budget = ctx->cache_budget;
    ctx->cache_budget = 0;  // the plan's own budget holds
    Plan *made = flat_in_reserve(ctx, &d);
    ctx->cache_budget = budget;
    CHECK((made != nullptr) == (need <= bound), "U=%lld: no flat plan\n", (long long)d.stats.dag_nodes);
    if (!made) return;
    CHECK(made == &d.plan && d.other.split == dom.split, "the plans changed places\n");
    CHECK(same(made->code_host, flat.code_host) && same(made->fill_host, flat.fill_host) &&
              same(made->reduce_host, flat.reduce_host) && same(made->store_host, flat.store_host) &&
              same(made->ind_rows_host, flat.ind_rows_host),
          "U=%lld: another flat plan\n", (long long)d.stats.dag_nodes);
    CHECK((char *)(made->ind_rows_dev + made->ind_rows_host.size()) <= block.data() + bound, "past the block\n");
    CHECK(flat_in_reserve(ctx, &d) == nullptr, "made twice\n");
}

}  // namespace

int main() {
    tgp_ctx_s c;
    c.plan_upload = false;
    c.cache_budget = (size_t)72 << 30;
    {   // 32-bit offsets: 18000 entries of 4 KiB and of 512 KiB
        tgp_dag_s d;
        column_trees(d, &c, 18000);
        const tgp_domain_s a = domain(&c, {1024, 1024}), b = domain(&c, {8, 131072}), line = domain(&c, {1 << 20});
        use(&c, d, a);
        CHECK(d.plan.split == 1 && d.plan.n_tab[1] == 18000, "1024 x 1024: no tables\n");
        const uint2 *code = d.plan.code_host.data();
        for (int i = 0; i < 3; ++i) {
            use(&c, d, b);
            CHECK(d.plan.split == 0, "8 x 131072: tables\n");
            CHECK(d.other.code_host.data() == code, "the plan with tables moved\n");
            use(&c, d, a);
            CHECK(d.plan.split == 1 && d.plan.code_host.data() == code, "1024 x 1024: planned again\n");
            use(&c, d, line);
            CHECK(d.plan.split == 0, "a line: tables\n");
        }
        CHECK(g_planned == 2, "planned %d times\n", g_planned);
        // another number of cases takes the place of both
        use(&c, d, domain(&c, {512, 1024}));
        CHECK(d.plan.split == 1 && d.other.cases < 0, "plans of another size kept\n");
    }
    {   // a column table of 8191 entries of 512 KiB is within the offsets, one of 8192 is not
        const tgp_domain_s b = domain(&c, {8, 131072});
        for (int n : {8191, 8192}) {
            tgp_dag_s d;
            column_trees(d, &c, n);
            for (int i = 0; i < 2; ++i) {
                use(&c, d, domain(&c, {1024, 1024}));
                CHECK(d.plan.split == 1, "%d entries of 4 KiB: no tables\n", n);
                use(&c, d, b);
                CHECK((d.plan.split == 1) == (n == 8191), "%d entries of 512 KiB: split %d\n", n, d.plan.split);
            }
        }
        g_planned = 0;
    }
    {   // the order does not matter: refused where they do not fit, planned where they do
        tgp_dag_s d;
        column_trees(d, &c, 18000);
        g_planned = 0;
        for (int i = 0; i < 3; ++i) {
            use(&c, d, domain(&c, {8, 131072}));
            CHECK(d.plan.split == 0, "8 x 131072 first: tables\n");
            use(&c, d, domain(&c, {1024, 1024}));
            CHECK(d.plan.split == 1, "1024 x 1024 second: no tables\n");
        }
        CHECK(g_planned == 2, "planned %d times\n", g_planned);
    }
    {   // a flat plan first; tables that cannot be planned beside it are not tried twice
        tgp_dag_s d;
        column_trees(d, &c, 18000);
        g_planned = 0;
        use(&c, d, domain(&c, {1 << 20}));
        for (int i = 0; i < 3; ++i) {
            use(&c, d, domain(&c, {8, 131072}));
            CHECK(d.plan.split == 0 && d.other.cases < 0, "8 x 131072: tables\n");
        }
        CHECK(g_planned == 2, "planned %d times\n", g_planned);
    }
    {   // the budget: half of it holds the tables of 64 x 64, not those of 8 x 512
        tgp_dag_s d;
        column_trees(d, &c, 100);
        g_planned = 0;
        c.cache_budget = 8 * 4 * 4096;
        for (int i = 0; i < 3; ++i)
            for (auto &s : {std::vector<int64_t>{64, 64}, {8, 512}, {32, 128}, {128, 32}, {4096}, {16, 16, 16}}) {
                use(&c, d, domain(&c, s));
                const bool fits = s.size() == 2 && s[1] <= 128;
                CHECK((d.plan.split > 0) == fits, "%lld..: split %d\n", (long long)s[0], d.plan.split);
            }
        CHECK(g_planned == 2, "planned %d times\n", g_planned);
    }
    c.plan_upload = true;
    c.cache_budget = (size_t)72 << 30;
    Gen g(20261206);
    for (int i = 0; i < 12; ++i) {
        check_reserve(&c, g, 20 + 5 * i, 1, 5 + i % 4, domain(&c, {64, 64}));
        check_reserve(&c, g, 200, 1 + i % 3, 4 + i % 6, domain(&c, {33, 127}));
        check_reserve(&c, g, 1, 1, 1 + i, domain(&c, {8, 128}));
    }
    check_reserve(&c, g, 2500, 3, 11, domain(&c, {32, 32}));  // planned by several threads
    if (g_bad) {
        printf("%d failures\n", g_bad);
        return 1;
    }
    printf("OK\n");
    return 0;
}
