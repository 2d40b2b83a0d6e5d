// Host check of the planning threads (runtime.cpp, compiled for the CPU as in
// planner_check.cpp; no device call): in a process that gets no more threads, a
// team has the ones that could be made, and a large DAG is planned as with all
// of them.
#define main planner_check_main
#include "planner_check.cpp"
#undef main

#include <sys/resource.h>

int main() {
    Gen g(7);
    tgp_dag_s d;
    make_dag(d, g, 2500, 3, 11);
    CHECK(d.stats.dag_nodes >= kParallelDecideNodes, "%lld nodes\n", (long long)d.stats.dag_nodes);
    std::vector<uint2> code[2];
    int32_t slots[2];
    auto plan = [&](HostTeam &team, int i) {
        d.plan = Plan();
        PlanJob w(&d, 4096, 8, (size_t)1 << 24);
        w.pl.team = &team;
        plan_prepare(w, false, 8);
        CHECK(plan_decide_emit(w, 8, true, 20.0, 0, 8) == TGP_OK, "plan\n");
        code[i] = d.plan.code_host;
        slots[i] = d.plan.n_slots;
    };
    HostTeam all;
    plan(all, 0);
    // room for two or three more stacks
    FILE *f = fopen("/proc/self/statm", "r");
    unsigned long pages = 0;
    CHECK(f && fscanf(f, "%lu", &pages) == 1, "statm\n");
    fclose(f);
    const size_t stack = (size_t)256 << 20, used = (size_t)pages * 4096;
    pthread_attr_t attr;
    pthread_attr_init(&attr);
    pthread_attr_setstacksize(&attr, stack);
    CHECK(pthread_setattr_default_np(&attr) == 0, "stack size\n");
    rlimit old;
    CHECK(getrlimit(RLIMIT_AS, &old) == 0, "limit\n");
    const rlimit lim{used + stack * 5 / 2, old.rlim_max};
    CHECK(setrlimit(RLIMIT_AS, &lim) == 0, "limit\n");
    HostTeam few;
    const int n = few.grow(16);
    CHECK(setrlimit(RLIMIT_AS, &old) == 0, "limit\n");
    printf("%d threads of 16\n", n);
    CHECK(n >= 2 && n < 16, "%d threads\n", n);
    std::atomic<int> ran{0};
    few.run(n, [&](int) { ++ran; });
    CHECK(ran == n, "%d of %d ran\n", ran.load(), n);
    plan(few, 1);
    CHECK(slots[0] == slots[1], "another plan\n");
    CHECK(code[0].size() == code[1].size() && memcmp(code[0].data(), code[1].data(), 8 * code[0].size()) == 0,
          "another plan\n");
    if (g_bad) {
        printf("%d failures\n", g_bad);
        return 1;
    }
    printf("OK\n");
    return 0;
}
