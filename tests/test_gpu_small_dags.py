"""Small DAGs on both sides of the line below which no tables are made: the
route is the one the line gives, and values and fitness are those of flat
programs, bit for bit."""
import numpy as np
import pytest

from paper_2103_07512_amd import popgen as pg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2103_07512_amd import tgp
    assert torch.cuda.is_available()
    return tgp, tgp.Context(0), torch


# trees, shape, tables: 2 + 3 x trees nodes; the line is 100 nodes and 2^25 node-evals
@pytest.mark.parametrize("trees,shape,tables", [(1, (64, 64), False), (32, (64, 64), False), (33, (64, 64), True),
                                                (32, (512, 668), False), (32, (512, 669), True), (1, (2560, 2570), False),
                                                (1, (2600, 2600), True)])
def test_line(env, trees, shape, tables):
    tgp, ctx, torch = env
    pop = pg.population_from_texts([f"add(mult(x, {0.01 * (i + 1):.2f}), y)" for i in range(trees)])
    dom, dag = tgp.Domain(ctx, shape), tgp.build_dag(ctx, pop)
    print(trees, shape, dag.stats()["dag_nodes"], "nodes", flush=True)
    t = torch.linspace(-1, 1, dom.cases, device="cuda:0").reshape(1, -1).contiguous()
    f, g = (torch.full((trees,), -1.0, dtype=torch.float64, device="cuda:0") for _ in range(2))
    v, w = (torch.full((trees, dom.cases), 7.0, dtype=torch.float32, device="cuda:0") for _ in range(2))
    tgp.fitness(ctx, dag, dom, t, tgp.RMSE, f)
    assert (ctx.last_work()["cached_nodes"] > 0) == tables
    tgp.evaluate(ctx, dag, dom, v)
    ctx.set_plan(cache_access_cost=-1.0)   # nothing cached: flat
    try:
        flat = tgp.build_dag(ctx, pop)
        tgp.fitness(ctx, flat, dom, t, tgp.RMSE, g)
        tgp.evaluate(ctx, flat, dom, w)
    finally:
        ctx.set_plan()
    torch.cuda.synchronize()
    assert torch.equal(v.view(torch.int32), w.view(torch.int32))
    assert torch.equal(f.view(torch.int64), g.view(torch.int64))
