"""Batches whose steps hold flat, wide and ragged jobs in turn and together, on
both sides of the lines where the forms are joined: every job of every run is
written, and equals the plain call bit for bit.  The graph is built again only
when a step has a form or level that none had before."""

import numpy as np
import pytest

from paper_2103_07512_amd import popgen as pg

pytestmark = pytest.mark.gpu

FUNCS = tuple(n for n, a in pg.OPS if a > 0 and n not in ("or", "xor", "and", "warp"))
ALL = tuple(n for n, a in pg.OPS if a > 0)
# name -> shapes; "large" holds more work items than small mixed batches are joined for
GROUPS = {"flat": [(1000,), (37,), (5, 7)], "image": [(40, 48)], "wide": [(16, 256), (8, 512)],
          "ragged": [(32, 32), (33, 127), (9, 8, 15)], "large": [(600, 512), (900,), (301, 203)]}


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2103_07512_amd import tgp
    assert torch.cuda.is_available()
    ctx = tgp.Context(0)
    ctx.set_tuning(4, 1)   # one split of the cases for the plain and the batched form
    jobs = {}
    for gi, (name, shapes) in enumerate(GROUPS.items()):
        jobs[name] = []
        for i, shape in enumerate(shapes):
            n = 130 if name == "large" else 12 + 5 * i
            # rewrites and operand-order hashing beside the plain DAGs
            ctx.set_hashing(commutative=(gi + i) % 3 == 1)
            ctx.set_rewrite((gi + i) % 3 == 2)
            pop = pg.ramped_half_and_half(n, 2, 5 + (gi + i) % 3, 1400 + 10 * gi + i, ALL if name == "image" else FUNCS,
                                          len(shape), 1)
            dom, dag = tgp.Domain(ctx, shape), tgp.build_dag(ctx, pop)
            fresh = tgp.build_dag(ctx, pop)
            rng = np.random.RandomState(gi * 10 + i)
            t = torch.from_numpy(rng.uniform(-1, 1, (1, dom.cases)).astype(np.float32)).to("cuda:0")
            out, ref = (torch.full((n,), -1.0, dtype=torch.float64, device="cuda:0") for _ in range(2))
            tgp.fitness(ctx, fresh, dom, t, tgp.RMSE, ref)
            torch.cuda.synchronize()
            jobs[name].append(((dag, dom, t, tgp.RMSE, out), ref.cpu().numpy().view(np.uint64)))
    ctx.set_hashing(commutative=False)
    ctx.set_rewrite(False)
    return tgp, ctx, torch, jobs


ORDER = [("flat",), ("flat",), ("wide",), ("ragged",), ("flat", "wide"), ("large",), ("image",), ("large", "wide", "ragged"),
         ("flat",), ("image", "wide"), ("wide",), ("large", "flat")]


@pytest.mark.parametrize("persistent", [True, False], ids=["persistent", "direct"])
@pytest.mark.parametrize("graph", [True, False], ids=["graph", "queued"])
def test_forms_in_turn(env, persistent, graph):
    tgp, ctx, torch, jobs = env
    ctx.set_batch_form(persistent)
    try:
        b = tgp.Batch(ctx, use_graph=graph)
        captures = []
        for rep in range(2):
            for names in ORDER:
                step = [j for n in names for j in jobs[n]]
                for (_, _, _, _, out), _ in step:
                    out.fill_(-1.0)
                b.run([j for j, _ in step])
                torch.cuda.synchronize()
                say(names, b.stats()["captures"])
                for (_, _, _, _, out), want in step:
                    np.testing.assert_array_equal(out.cpu().numpy().view(np.uint64), want)
                captures.append(b.stats()["captures"])
        if graph:
            assert captures[0] == captures[1] == 1
        else:
            assert captures[-1] == 0
    finally:
        ctx.set_batch_form(True)


def test_one_dag_on_two_shapes(env):
    tgp, ctx, torch, _ = env
    pop = pg.ramped_half_and_half(25, 2, 6, 1490, FUNCS, 2, 1)
    dag = tgp.build_dag(ctx, pop)
    step, want = [], []
    for i, shape in enumerate([(32, 64), (64, 40), (40, 64), (8, 256)]):
        dom = tgp.Domain(ctx, shape)
        t = torch.linspace(-1, 1, dom.cases, device="cuda:0").reshape(1, -1).contiguous()
        ref = torch.full((25,), -1.0, dtype=torch.float64, device="cuda:0")
        tgp.fitness(ctx, tgp.build_dag(ctx, pop), dom, t, tgp.MSE, ref)
        step.append((dag, dom, t, tgp.MSE, torch.full_like(ref, -1.0)))
        want.append(ref)
    torch.cuda.synchronize()
    b = tgp.Batch(ctx)
    for some in ([0], [0, 1], [1, 2], [2], [0, 1, 2, 3], [3]):
        for j in step:
            j[4].fill_(-1.0)
        b.run([step[i] for i in some])
        torch.cuda.synchronize()
        say("shapes", some)
        for i in some:
            np.testing.assert_array_equal(step[i][4].cpu().numpy().view(np.uint64), want[i].cpu().numpy().view(np.uint64))
