"""DAG builds whose levels hold 1023, 1024 or 1025 tokens each, around the line up
to which one launch takes all the upper levels, with fewer trees going on above,
against the oracle's DAG."""
import pytest

import oracle
from paper_2103_07512_amd import popgen as pg

from test_gpu_dag_sizes import env  # noqa: F401
from test_gpu_parity import _dag_equal

pytestmark = pytest.mark.gpu


def trees(n, taller):
    """n unary chains of seven operators over constants and axes (every third
    one a copy of an earlier), the first `taller` of them with nine more."""
    out = []
    for i in range(n):
        leaf = (pg.VAR, i % 2, 0.0) if i % 5 == 0 else (pg.CONST, 0, float(i - 3 if i % 3 == 0 else i))
        ops = ("sin", "abs", "neg", "cos", "sqrt", "neg", "sin") + (("exp", "neg", "sin") * 3 if i < taller else ())
        out.append(pg.make_tokens([leaf] + [(pg.OP_CODE[o], 0, 0.0) for o in ops]))
    return pg.Population.from_trees(out)


@pytest.mark.parametrize("n", [1023, 1024, 1025, 2049])
@pytest.mark.parametrize("taller", [0, 1, 65, 1023])
def test_level_sizes(env, n, taller):  # noqa: F811
    tgp, ctx, torch = env
    pop = trees(n, taller)
    print("levels", n, taller, len(pop.tokens), "tokens", flush=True)
    want = oracle.build_dag(pop.tokens, pop.offsets)
    _dag_equal(tgp.build_dag(ctx, pop).export(), want, "launch and rest")
    ctx.set_rewrite(True)
    try:
        _dag_equal(tgp.build_dag(ctx, pop).export(), oracle.build_dag(pop.tokens, pop.offsets, rewrite=True), "rewrites")
    finally:
        ctx.set_rewrite(False)
