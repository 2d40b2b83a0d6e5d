"""Constant folding in one launch (up to 2048 variable-free operator nodes of at
most 1024 heights) and past either limit: per-case values bitwise those of
programs that evaluate every constant subtree, and the folded count."""
import numpy as np
import pytest

from paper_2103_07512_amd import popgen as pg

from test_gpu_parity import env, gpu_eval  # noqa: F401

pytestmark = pytest.mark.gpu

BINARY = ("add", "sub", "mult", "div", "min", "max", "pow", "mod", "mdist", "len")


def op(name):
    return (pg.OP_CODE[name], 0, 0.0)


def const(v):
    return (pg.CONST, 0, v)


def used(tokens):
    """x + tokens: the constant subtree is an operand of a variable node."""
    return [(pg.VAR, 0, 0.0)] + tokens + [op("add")]


def singles(n):
    """n trees, each with one folded operator node of its own."""
    return [used([const(0.25 + i), const(1.0 + 0.001 * i), op(BINARY[i % len(BINARY)])]) for i in range(n)]


def comb(n):
    """One tree of n folded operator nodes, one of each height."""
    toks = [const(0.5)]
    for i in range(n):
        toks += [const(0.75 + 0.001 * i), op(("add", "mdist", "min", "sub")[i % 4])]
    return [used(toks)]


def mixed(seed):
    """Constant trees of every operator, NaN and infinite constants among them."""
    rng = pg.Rng(seed)
    mk = pg.TreeMaker(rng, tuple(n for n, a in pg.OPS if a > 0), 2)
    trees = []
    for i in range(40):
        toks = [(t["op"], t["var"], float(t["value"])) for t in mk.tree(2 + i % 5, True)]
        fill = (float("nan"), float("inf"), -0.0, 0.3, 1.5, -2.0, 0.25)
        trees.append(used([const(fill[(i + j) % 7]) if t[0] == pg.VAR else t for j, t in enumerate(toks)]))
    return trees


@pytest.mark.parametrize("name,trees", [
    ("one", singles(1)), ("1023", singles(1023)), ("1025", singles(1025)), ("2047", singles(2047)),
    ("2048", singles(2048)), ("2049", singles(2049)), ("tall 3", comb(3)), ("tall 1022", comb(1022)),
    ("tall 1023", comb(1023)), ("tall 1024", comb(1024)), ("tall 1025", comb(1025)), ("mixed", mixed(5))])
def test_fold_sizes(env, name, trees):  # noqa: F811
    tgp, ctx, torch = env
    pop = pg.Population.from_trees([pg.make_tokens(t) for t in trees])
    print("fold", name, pop.n_roots, "trees", flush=True)
    res = {}
    try:
        for on in (False, True):
            ctx.set_folding(on)
            got = gpu_eval(env, pop, (5, 7))[0]
            res[on] = (got, ctx.last_work()["folded_nodes"])
    finally:
        ctx.set_folding(True)
    a, b = res[False][0], res[True][0]
    assert res[False][1] == 0 and res[True][1] > 0
    if not name.startswith("mixed"):
        assert res[True][1] == len(trees)
    assert np.array_equal(np.isnan(a), np.isnan(b))
    m = ~np.isnan(a)
    assert np.array_equal(a[m].view(np.uint32), b[m].view(np.uint32))
