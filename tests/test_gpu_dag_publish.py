"""Populations whose DAG block, sized for as many nodes as tokens, lies on either
side of the 8 MB that the build writes to the staging itself, against the
oracle's DAG."""
import pytest

import oracle

from test_gpu_dag_sizes import env, population  # noqa: F401
from test_gpu_parity import _dag_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("total,whole", [(255000, True), (265000, False)])
def test_block_sizes(env, total, whole):  # noqa: F811
    tgp, ctx, torch = env
    pop = population(total, total)
    assert (8192 + 4 * (8 * total + pop.n_roots) <= 8 << 20) == whole
    print("block", total, pop.n_roots, "trees", flush=True)
    _dag_equal(tgp.build_dag(ctx, pop).export(), oracle.build_dag(pop.tokens, pop.offsets), "host tokens")
