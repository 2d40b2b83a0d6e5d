"""Device memory of DAGs that are kept: a converged population's DAG holds
memory for its nodes, not for its tokens."""
import numpy as np
import pytest

import oracle
from paper_2103_07512_amd import popgen as pg

from test_gpu_parity import _dag_equal

pytestmark = pytest.mark.gpu


# tokens: read back with a copy of their own, and published by the build
@pytest.mark.parametrize("tokens", [500_000, 200_000])
def test_kept_dags(tokens):
    import torch
    from paper_2103_07512_amd import tgp
    ctx = tgp.Context(0)
    some = pg.ramped_half_and_half(120, 2, 8, 77, pg.F18, 2)
    reps = -(-tokens // len(some.tokens))
    off = np.concatenate([[0]] + [some.offsets[1:] + i * len(some.tokens) for i in range(reps)]).astype(np.int64)
    pop = pg.Population(tokens=np.tile(some.tokens, reps), offsets=off, n_individuals=120 * reps, n_channels=1)
    dags, free = [], []
    for i in range(9):
        dags.append(tgp.build_dag(ctx, pop))
        torch.cuda.synchronize()
        free.append(torch.cuda.mem_get_info()[0])
    st = dags[0].stats()
    held = (free[1] - free[8]) / 7
    print(len(pop.tokens), "tokens", st["dag_nodes"], "nodes", held, "bytes a DAG", flush=True)
    assert st["dag_nodes"] * 20 < len(pop.tokens)
    assert held <= 2 * 4 * (8 * st["dag_nodes"] + pop.n_roots) + (2 << 20)
    assert held < 16 * len(pop.tokens)
    want = oracle.build_dag(pop.tokens, pop.offsets)
    for d in (dags[0], dags[8]):
        _dag_equal(d.export(), want, "kept")
    # the constants are folded from the device's arrays
    dom = tgp.Domain(ctx, (40, 56))
    t = torch.linspace(-1, 1, dom.cases, device="cuda:0").reshape(1, -1).contiguous()
    out = np.empty(pop.n_individuals)
    ref = np.empty(120)
    tgp.fitness(ctx, dags[0], dom, t, tgp.RMSE, out)
    tgp.fitness(ctx, tgp.build_dag(ctx, some), dom, t, tgp.RMSE, ref)
    np.testing.assert_array_equal(out.view(np.uint64), np.tile(ref, reps).view(np.uint64))
