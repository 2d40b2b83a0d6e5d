"""The wave-wide tree scan (children, heights, sizes and depths, 64 tokens at a
time): trees whose lengths and stack depths straddle the scan's limits, against
the oracle's DAG and breeding, and the first error of a malformed tree."""
import numpy as np
import pytest

import oracle
from paper_2103_07512_amd import popgen as pg

from test_gpu_breed import _check, env  # noqa: F401  (env: the module's fixture)
from test_gpu_parity import _dag_equal

pytestmark = pytest.mark.gpu


def right_comb(n, op, arity):
    """n nested operators, every operand but the last a leaf: the postfix
    stack grows to 1 + n (arity - 1)."""
    toks = []
    for i in range(n):
        toks += [(pg.VAR, i % 2, 0.0)] * (arity - 1)
    toks.append((pg.CONST, 0, 0.25 + n))
    return toks + [(pg.OP_CODE[op], 0, 0.0)] * n


def left_comb(n, op):
    toks = [(pg.CONST, 0, 0.5 + n)]
    for i in range(n):
        toks += [(pg.VAR, i % 2, 0.0), (pg.OP_CODE[op], 0, 0.0)]
    return toks


def chain(n, ops=("sin", "abs", "neg")):
    return [(pg.VAR, 0, 0.0)] + [(pg.OP_CODE[ops[i % len(ops)]], 0, 0.0) for i in range(n)]


def edge_population():
    trees = []
    for n in (0, 1, 62, 63, 64, 65, 126, 127, 128, 129, 200):
        trees.append(chain(n))
    for n in (1, 31, 32, 33, 63, 64, 65, 100):
        trees += [right_comb(n, "add", 2), left_comb(n, "sub"), right_comb(n, "clip", 3)]
    for n in (254, 255, 256, 257, 300, 700):   # around and past the table's 256 slots
        trees.append(right_comb(n, "add", 2))
    trees += [right_comb(128, "if", 3), right_comb(200, "lerp", 3)]
    rng = pg.Rng(77)
    mk = pg.TreeMaker(rng, pg.F18 + ("lerp", "if"), 2)
    out = [pg.make_tokens(t) for t in trees] + [mk.tree(d, full) for d in (3, 7, 10) for full in (True, False) for _ in range(4)]
    return pg.Population.from_trees(out)


def test_scan_limits_dag(env):  # noqa: F811
    tgp, ctx, torch = env
    pop = edge_population()
    print("scan limits:", pop.n_roots, "trees", flush=True)
    _dag_equal(tgp.build_dag(ctx, pop).export(), oracle.build_dag(pop.tokens, pop.offsets), "scan limits")


def test_scan_limits_breed(env):  # noqa: F811
    pop = edge_population()
    fit = np.random.RandomState(3).rand(pop.n_individuals)
    _check(env, pop, fit, 5, 120, functions=[pg.OP_CODE[f] for f in pg.F18], max_depth=400)


@pytest.mark.parametrize("first", ["parse", "op"])
@pytest.mark.parametrize("at", [1, 63, 64, 130])
def test_first_error_wins(env, first, at):  # noqa: F811
    """An operand missing at one token and an unknown operator at a later one,
    or the other way round: the earlier one is reported."""
    tgp, ctx, torch = env
    toks = pg.make_tokens(chain(200))
    miss, unknown = (at, at + 40) if first == "parse" else (at + 40, at)
    toks[miss]["op"] = pg.OP_CODE["add"]
    toks[unknown]["op"] = 99
    good = pg.make_tokens(chain(3))
    all_toks = np.concatenate([good, toks])
    with pytest.raises(tgp.TgpError) as e:
        tgp.Dag(ctx, all_toks, np.array([0, 4, len(all_toks)]), 2)
    assert e.value.status == (-2 if first == "parse" else -4) and "tree 1" in str(e.value)
