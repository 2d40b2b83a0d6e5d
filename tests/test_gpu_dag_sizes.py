"""The DAG build's two ways -- one workgroup for small populations, a launch
per level for others -- at the sizes where they meet, and with trees taller
than the level counters, against the oracle's DAG; host and device tokens."""
import numpy as np
import pytest

import oracle
from paper_2103_07512_amd import popgen as pg

from test_gpu_parity import _dag_equal

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2103_07512_amd import tgp
    assert torch.cuda.is_available()
    return tgp, tgp.Context(0), torch


def chain(n, v=0):
    return pg.make_tokens([(pg.VAR, v, 0.0)] + [(pg.OP_CODE[("sin", "abs", "neg")[i % 3]], 0, 0.0) for i in range(n)])


def population(total, seed, tall=0):
    """Random trees (shared constants among them) of `total` tokens in all."""
    mk = pg.TreeMaker(pg.Rng(seed), pg.F18, 2)
    trees, n = ([chain(tall)], tall + 1) if tall else ([], 0)
    while n < total:
        t = mk.tree(2 + len(trees) % 7, len(trees) % 2 == 0)
        if n + len(t) > total:
            t = chain(total - n - 1, len(trees) % 2)
        t["value"][(t["op"] == 1) & (np.arange(len(t)) % 3 == 0)] = 0.5
        trees.append(t)
        n += len(t)
    return pg.Population.from_trees(trees)


@pytest.mark.parametrize("total,tall", [(1, 0), (64, 0), (1023, 0), (1024, 0), (1025, 0), (6143, 0), (6144, 0),
                                        (6145, 0), (20000, 0), (3000, 511), (3000, 512), (3000, 700), (9000, 511),
                                        (9000, 512)])
def test_build_ways(env, total, tall):
    tgp, ctx, torch = env
    pop = population(total, 11 + total, tall)
    assert len(pop.tokens) == total
    print("build", total, tall, pop.n_roots, "trees", flush=True)
    want = oracle.build_dag(pop.tokens, pop.offsets)
    _dag_equal(tgp.build_dag(ctx, pop).export(), want, "host tokens")
    tok = torch.from_numpy(pop.tokens.view(np.uint8).copy()).to("cuda:0")
    off = torch.from_numpy(pop.offsets.copy()).to("cuda:0")
    _dag_equal(tgp.Dag(ctx, tok, off, pop.n_individuals).export(), want, "device tokens")
    tgp.debug_set_hash_bits(3)
    try:
        if total <= 3000:
            _dag_equal(tgp.build_dag(ctx, pop).export(), want, "colliding hashes")
    finally:
        tgp.debug_set_hash_bits(0)


def test_bad_device_offsets(env):
    tgp, ctx, torch = env
    tok = torch.from_numpy(chain(9).view(np.uint8).copy()).to("cuda:0")
    for offsets in ([1, 10], [0, -1], [0, 1 << 40]):
        off = torch.tensor(offsets, dtype=torch.int64, device="cuda:0")
        with pytest.raises(tgp.TgpError) as e:
            tgp.Dag(ctx, tok, off, 1)
        assert e.value.status == -1
    off = torch.tensor([0, 0, 0], dtype=torch.int64, device="cuda:0")
    with pytest.raises(tgp.TgpError) as e:
        tgp.Dag(ctx, tok, off, 2)
    assert e.value.status == -2 and "tree 0" in str(e.value)
    off = torch.tensor([0, 12, 10], dtype=torch.int64, device="cuda:0")  # decreasing past the end
    with pytest.raises(tgp.TgpError) as e:
        tgp.Dag(ctx, tok, off, 2)
    assert e.value.status == -1 and "tree 0" in str(e.value)
