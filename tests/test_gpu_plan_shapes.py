"""One DAG evaluated on several grid shapes of one number of cases: every call
gives the bits of a fresh DAG on that shape, whichever shapes came before, in
the plain, rendering, no-allocation and batched forms, with and without a
cache budget that holds the tables of some of the shapes only."""

import numpy as np
import pytest

from paper_2103_07512_amd import popgen as pg

pytestmark = pytest.mark.gpu

FUNCS = tuple(n for n, a in pg.OPS if a > 0 and n not in ("or", "xor", "and", "warp"))
PLANE = [(64, 64), (8, 512), (512, 8), (16, 256), (16, 16, 16), (2, 2048)]
LINE = [(4096,), (64, 64), (8, 512), (1, 4096), (4096, 1)]


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2103_07512_amd import tgp
    assert torch.cuda.is_available()
    return tgp, tgp.Context(0), torch


def _bits(t):
    return t.cpu().numpy().view(np.uint64)


@pytest.mark.parametrize("axes,shapes", [(2, PLANE), (1, LINE)], ids=["plane", "line"])
@pytest.mark.parametrize("budget", [1 << 36, 4 * 4 * 4096], ids=["large", "small"])
def test_shapes_in_turn(env, axes, shapes, budget):
    tgp, ctx, torch = env
    # few subtrees are shared, so that a small budget is one for tables
    pop = pg.ramped_half_and_half(24, 2, 5, 1200 + axes, FUNCS, axes, 1)
    ctx.set_cache_budget(budget)
    try:
        dag = tgp.build_dag(ctx, pop)
        rng = np.random.RandomState(7)
        t = torch.from_numpy(rng.uniform(-1, 1, (1, 4096)).astype(np.float32)).to("cuda:0")
        want, doms, cached = [], [], []
        for s in shapes:
            dom = tgp.Domain(ctx, s)
            fresh = tgp.build_dag(ctx, pop)
            f = torch.full((pop.n_individuals,), -1.0, dtype=torch.float64, device="cuda:0")
            v = torch.full((pop.n_roots, 4096), 7.0, dtype=torch.float32, device="cuda:0")
            tgp.fitness(ctx, fresh, dom, t, tgp.RMSE, f)
            cached.append(ctx.last_work()["cached_nodes"])
            tgp.evaluate(ctx, fresh, dom, v)
            torch.cuda.synchronize()
            want.append((_bits(f), v.cpu().numpy()))
            doms.append(dom)
        say("cached nodes", dict(zip(shapes, cached)))
        if budget < 1 << 30 and axes == 2:
            assert cached[0] != cached[1], "one budget was to hold the tables of the first shape only"
        order = list(range(len(shapes))) + list(range(len(shapes)))[::-1]
        for i in order:
            say("shape", shapes[i])
            o = torch.full((3, pop.n_individuals), -1.0, dtype=torch.float64, device="cuda:0")
            v = torch.full((pop.n_roots, 4096), 7.0, dtype=torch.float32, device="cuda:0")
            tgp.fitness(ctx, dag, doms[i], t, tgp.RMSE, o[0])
            tgp.evaluate(ctx, dag, doms[i], v)
            tgp.fitness_noalloc(ctx, dag, doms[i], t, tgp.RMSE, o[1])
            tgp.fitness_batch(ctx, [(dag, doms[i], t, tgp.RMSE, o[2])])
            torch.cuda.synchronize()
            np.testing.assert_array_equal(_bits(o[0]), want[i][0])
            np.testing.assert_array_equal(_bits(o[1]), want[i][0])
            np.testing.assert_allclose(o[2].cpu().numpy(), want[i][0].view(np.float64), rtol=1e-6)
            a, b = v.cpu().numpy(), want[i][1]
            assert np.array_equal(np.isnan(a), np.isnan(b))
            m = ~np.isnan(a)
            assert np.array_equal(a[m].view(np.uint32), b[m].view(np.uint32))
    finally:
        ctx.set_cache_budget(1 << 36)
