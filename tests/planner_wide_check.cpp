// Host check of wide plans (runtime.cpp, compiled for the CPU as in
// planner_check.cpp, whose random DAGs and stack machine it uses; no device
// call).  Random populations over two and three axes are planned with their
// axes split into grid rows and columns, sequentially and level-parallel, and
// every emitted program is run on the host stack machine:
//   - the tables' programs, level by level, give bit for bit the value of
//     direct evaluation of their node, reading only entries of lower levels;
//   - so do the fill, reduce and store programs, which read the tables;
//   - table entries depend on one side of the split only, and every other
//     subtree a program reads has variables on both sides;
//   - both decision passes cache the same nodes at the same levels when they
//     spill the same;
//   - a budget without room for the tables gives the flat plan of the same DAG.
#define main planner_check_main
#include "planner_check.cpp"
#undef main

namespace {

int64_t g_pairs = 0;

// The plan with its table operands turned into cache reads: the cache rows
// are followed by the row table's entries, then the column table's.  A pair
// form becomes two instructions, so the programs move: their descriptors are
// translated too.
Plan with_tables_as_rows(const Plan &P) {
    Plan Q;
    Q.fill_host = P.fill_host;
    Q.reduce_host = P.reduce_host;
    Q.store_host = P.store_host;
    const uint32_t at[2] = {(uint32_t)P.n_slots, (uint32_t)(P.n_slots + P.n_tab[0])};
    std::vector<uint32_t> moved(P.code_host.size() + 1);
    for (size_t i = 0; i < P.code_host.size(); ++i) {
        moved[i] = (uint32_t)Q.code_host.size();
        const uint2 w = P.code_host[i];
        const uint32_t c = w.x & 0xffu, S = w.x >> 8;
        if (i >= (size_t)P.tab_code_end && c >= kPairBase) {
            const uint32_t v = c - kPairBase, row = at[0] + (w.y & 0xffffu), col = at[1] + (w.y >> 16);
            ++g_pairs;
            // push one operand, the fused form reads the other as the last child
            Q.code_host.push_back(uint2{(S << 8) | I_CACHE, row});
            Q.code_host.push_back(uint2{((S + 1) << 8) | (kFuseBase + 16 * kFuseCache + v), col});
            continue;
        }
        Q.code_host.push_back(w);
    }
    moved[P.code_host.size()] = (uint32_t)Q.code_host.size();
    for (auto *list : {&Q.fill_host, &Q.reduce_host, &Q.store_host})
        for (ProgDesc &pd : *list) {
            const uint32_t end = moved[pd.code_off + pd.len];
            pd.code_off = moved[pd.code_off];
            pd.len = end - pd.code_off;
        }
    for (size_t i = moved[P.tab_code_end]; i < Q.code_host.size(); ++i) {
        uint2 &ins = Q.code_host[i];
        const uint32_t c = ins.x & 0xffu;
        if (c == I_X || c == I_Y) {
            ins.y += at[c == I_X ? 0 : 1];
            ins.x = (ins.x & ~0xffu) | I_CACHE;
        } else if (c >= kFuseBase && c < kFuseBase + 32) {
            const uint32_t kind = (c - kFuseBase) / 16;
            ins.y += at[kind];
            ins.x += 16 * (kFuseCache - kind);
        }
    }
    return Q;
}

void check_wide(const char *what, tgp_dag_s &d, PlanJob &w, int D, int split, int ndim, Gen &g) {
    const Plan &P = d.plan;
    const Plan Q = with_tables_as_rows(P);
    const Planner &pl = w.pl;
    const int64_t U = d.stats.dag_nodes;
    std::vector<int32_t> node_of[2] = {std::vector<int32_t>(P.n_tab[0], -1), std::vector<int32_t>(P.n_tab[1], -1)};
    for (int64_t n = 0; n < U; ++n) {
        const bool tab = pl.cached[n] && pl.in_table(n);
        if (tab) node_of[pl.cls[n] - 1][pl.slot[n]] = (int32_t)n;
        CHECK(!(pl.cached[n] && !pl.in_table(n)) || pl.cls[n] == 3, "%s: cache row of a one-sided node\n", what);
    }
    for (int cs = 0; cs < 4; ++cs) {
        float v3[3];
        for (int k = 0; k < 3; ++k) v3[k] = cs == k ? 0.0f : (float)(g.u() * 4 - 2);
        std::vector<float> val(U);
        for (int64_t n = 0; n < U; ++n) {
            const int op = d.op[n] & 0xff;
            const int32_t *k = &d.kid[3 * n];
            if (op == TGP_VAR) val[n] = v3[(d.op[n] >> 8) & 0xff];
            else if (op == TGP_CONST) val[n] = d.value[n];
            else val[n] = apply(op, val[k[0]], k[1] >= 0 ? val[k[1]] : 0.0f, k[2] >= 0 ? val[k[2]] : 0.0f);
        }
        std::vector<float> tab[2] = {std::vector<float>(P.n_tab[0], NAN), std::vector<float>(P.n_tab[1], NAN)};
        std::vector<float> cache(P.n_slots, NAN);
        auto all = [&]() {
            std::vector<float> c(cache);
            c.insert(c.end(), tab[0].begin(), tab[0].end());
            c.insert(c.end(), tab[1].begin(), tab[1].end());
            return c;
        };
        for (int l = 0; l < P.levels(); ++l) {
            if (l < (int)P.tab_level.size())
                for (int32_t i = P.tab_level[l].first; i < P.tab_level[l].last; ++i) {
                    const ProgDesc &pd = P.tab_host[i];
                    const int t = i < P.tab_level[l].mid ? 0 : 1;
                    const float a = t ? v3[split] : v3[0], b = t ? (split + 1 < ndim ? v3[split + 1] : NAN) : v3[1];
                    std::vector<int32_t> reads;
                    float v;
                    const bool ok = run(P, pd, D, a, b, tab[t], &v, &reads);
                    CHECK(ok, "%s: table program %d malformed\n", what, i);
                    if (!ok) continue;
                    const int32_t node = node_of[t][pd.dest];
                    CHECK(pl.level[node] == l, "%s: entry at level %d, planned %d\n", what, l, pl.level[node]);
                    for (int32_t r : reads)
                        CHECK(pl.level[node_of[t][r]] < l, "%s: level %d reads a table entry of level %d\n", what, l,
                              pl.level[node_of[t][r]]);
                    CHECK(memcmp(&v, &val[node], 4) == 0, "%s: table entry of node %d gives %a, direct %a\n", what,
                          node, v, val[node]);
                    tab[t][pd.dest] = v;
                }
            if (l + 1 >= (int)P.level_first.size()) continue;
            for (int32_t i = P.level_first[l]; i < P.level_first[l + 1]; ++i) {
                const ProgDesc &pd = Q.fill_host[i];
                float v;
                const bool ok = run(Q, pd, D, NAN, NAN, all(), &v, nullptr);
                const int32_t node = P.slot_node[pd.dest];
                CHECK(ok && memcmp(&v, &val[node], 4) == 0, "%s: fill of node %d\n", what, node);
                cache[pd.dest] = v;
            }
        }
        const std::vector<float> c = all();
        for (int pass = 0; pass < 2; ++pass)
            for (const ProgDesc &pd : pass ? Q.store_host : Q.reduce_host) {
                float v;
                const bool ok = run(Q, pd, D, NAN, NAN, c, &v, nullptr);
                const int32_t node = pass ? d.roots[pd.dest] : w.reduce_list[pd.dest].first;
                CHECK(ok && memcmp(&v, &val[node], 4) == 0, "%s: root node %d\n", what, node);
            }
    }
}

}  // namespace

int main() {
    Gen g(20261205);
    struct Case {
        int n_ind, n_ch, d_max, D, ndim, split;
        double access;
    };
    const Case cases[] = {{40, 1, 6, 8, 2, 1, 20.0},   {60, 2, 9, 4, 3, 1, 20.0},   {60, 2, 9, 4, 3, 2, 2.0},
                          {300, 3, 10, 8, 2, 1, 2.0},  {2500, 3, 11, 8, 2, 1, 20.0}, {2500, 3, 12, 4, 3, 2, 20.0},
                          {2500, 1, 12, 3, 2, 1, 20.0}, {30, 1, 3, 8, 1, 1, 20.0}};
    for (const Case &c : cases) {
        tgp_dag_s d;
        make_dag(d, g, c.n_ind, c.n_ch, c.d_max);
        const int64_t U = d.stats.dag_nodes;
        // the axes: random_tree draws 0 or 1; spread them over three, or one
        for (int64_t n = 0; n < U; ++n)
            if ((d.op[n] & 0xff) == TGP_VAR) {
                const int v = c.ndim == 1 ? 0 : (c.ndim == 3 && n % 3 == 0 ? 2 : (d.op[n] >> 8) & 0xff);
                d.op[n] = TGP_VAR | v << 8;
            }
        std::vector<uint8_t> cached[2];
        std::vector<int32_t> level[2];
        int64_t spills[2] = {-1, -2};
        for (int threads : {1, 8}) {
            char what[160];
            snprintf(what, sizeof what, "U=%lld D=%d ndim=%d split=%d threads=%d", (long long)U, c.D, c.ndim, c.split,
                     threads);
            for (size_t budget : {(size_t)1 << 24, (size_t)0}) {
                d.plan = Plan();
                PlanJob w(&d, 65536, c.D, budget);
                w.pl.split = c.split;
                w.pl.slot_bytes = 4.0 * 65536;
                w.pl.table_slots_per[0] = w.pl.table_slots_per[1] = 1.0 / 256;
                plan_prepare(w, true);
                if (!w.pl.folded.empty()) {  // the folded subtrees' values (no variable: any case)
                    w.pl.fold_val.assign(U, 0.0f);
                    for (int64_t n = 0; n < U; ++n) {
                        const int op = d.op[n] & 0xff;
                        const int32_t *k = &d.kid[3 * n];
                        float *v = w.pl.fold_val.data();
                        v[n] = kArity[op] == 0 ? d.value[n]
                                               : apply(op, v[k[0]], k[1] >= 0 ? v[k[1]] : 0, k[2] >= 0 ? v[k[2]] : 0);
                    }
                }
                const tgp_status st = plan_decide_emit(w, c.D, true, c.access, 1, threads);
                if (!budget) {  // no room for tables (nor, perhaps, for the flat plan's spills)
                    CHECK(d.plan.tab_host.empty() && d.plan.split == 0, "%s: tables without a budget\n", what);
                    CHECK(st == TGP_OK || (st == TGP_ENOMEM && w.pl.spills > 0), "%s: status %d\n", what, st);
                    continue;
                }
                CHECK(st == TGP_OK && d.plan.split == c.split, "%s: status %d\n", what, st);
                if (st != TGP_OK) continue;
                check_wide(what, d, w, c.D, c.split, c.ndim, g);
                const int t = threads == 1 ? 0 : 1;
                spills[t] = w.pl.spills;
                cached[t] = w.pl.cached;
                level[t] = w.pl.level;
                printf("%s: rows %d row entries %d column entries %d table levels %zu levels %d spills %lld\n", what,
                       d.plan.n_slots, d.plan.n_tab[0], d.plan.n_tab[1], d.plan.tab_level.size(), d.plan.levels(),
                       (long long)w.pl.spills);
            }
        }
        if (spills[0] == spills[1])
            CHECK(cached[0] == cached[1] && level[0] == level[1], "U=%lld: passes differ\n", (long long)U);
    }
    printf("%lld pair forms\n", (long long)g_pairs);
    CHECK(g_pairs > 0, "no pair form emitted\n");
    if (g_bad) {
        printf("%d failures\n", g_bad);
        return 1;
    }
    printf("OK\n");
    return 0;
}
