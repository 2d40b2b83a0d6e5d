"""The tables of served requests lie in the server's cache memory: they wait for
room there like cached rows, and a request whose tables find none in one piece
is evaluated without them."""

import numpy as np
import pytest

from paper_2103_07512_amd import popgen as pg

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2103_07512_amd import tgp
    assert torch.cuda.is_available()
    return tgp, tgp.Context(0), torch


def _pairs(seed, n):
    """Trees of n one-sided pairs with constants of their own."""
    c = np.random.RandomState(seed).randint(1, 1 << 20, size=(8, n, 2)) / float(1 << 20)
    def tree(cs):
        parts = [f"mult(sin(mult(x, {a:.7f})), cos(mult(y, {b:.7f})))" for a, b in cs]
        while len(parts) > 1:
            parts = [f"add({parts[i]}, {parts[i + 1]})" if i + 1 < len(parts) else parts[i]
                     for i in range(0, len(parts), 2)]
        return parts[0]
    return pg.population_from_texts([tree(cs) for cs in c])


def _plain(env, pop, dom, t):
    tgp, ctx, torch = env
    ref = np.empty(pop.n_individuals)
    tgp.fitness(ctx, tgp.build_dag(ctx, pop), dom, t, tgp.MSE, ref)
    return ref


def test_tables_count_to_the_budget(env):
    tgp, ctx, torch = env
    # 8 trees of 128 pairs: 2048 entries of 8 KiB, 16.8 MB of tables a request
    dom = tgp.Domain(ctx, (2048, 2048))
    t = torch.zeros(1, dom.cases, dtype=torch.float32, device="cuda:0")
    pops = [_pairs(i, 128) for i in range(12)]
    want = [_plain(env, p, dom, t) for p in pops]
    srv = tgp.Server(ctx, cache_budget_bytes=72 << 20)
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for rep in range(2):
        keys = [srv.submit(i, p, dom, t, tgp.MSE) for i, p in enumerate(pops)]
        for k, w in zip(keys, want):
            np.testing.assert_allclose(srv.wait(k), w, rtol=1e-6)
    st = srv.stats()
    used = free0 - torch.cuda.mem_get_info()[0]
    say("peak", st["bytes_peak"], "of", st["bytes_capacity"], "most active", st["max_active_seen"], "beyond the cache", used)
    srv.close()
    assert st["failed"] == 0 and st["completed"] == 24
    assert 16 << 20 < st["bytes_peak"] <= st["bytes_capacity"]
    assert st["max_active_seen"] <= 4        # of 16.8 MB each in 72 MiB
    assert used < 64 << 20                   # 12 requests' tables: 201 MB


def test_no_room_in_one_piece(env):
    tgp, ctx, torch = env
    dom = tgp.Domain(ctx, (64, 64))          # rows of 16 KiB
    t = torch.zeros(1, dom.cases, dtype=torch.float32, device="cuda:0")

    def one_row(i):
        """Trees that share one costly subtree of both sides, and it alone."""
        s = f"pow(sin(exp(mult(x, y))), cos(add(x, {i}.5)))"
        return [f"add({s}, {0.125 * j + i:.3f})" for j in range(8)]
    srv = tgp.Server(ctx, cache_budget_bytes=17 * 16384)
    for i in range(16):                      # rows of the two runs in turn
        pop = pg.population_from_texts(one_row(i))
        k = srv.submit(i % 2, pop, dom, t, tgp.MSE)
        np.testing.assert_allclose(srv.wait(k), _plain(env, pop, dom, t), rtol=1e-6)
        assert srv.ticket_info(k)["cache_new"] == 1
    st = srv.stats()
    assert st["entries"] == 16 and st["evictions"] == 0, st
    srv.end_run(1)
    # reads the rows between the holes, with 200 one-sided subtrees: 51 KB of tables
    texts = [s for i in range(0, 16, 2) for s in one_row(i)[:2]]
    texts += [f"mult(sin(mult(x, 0.{i:03d})), cos(mult(y, 0.{i:03d})))" for i in range(101, 201)]
    pop = pg.population_from_texts(texts)
    k = srv.submit(0, pop, dom, t, tgp.MSE)
    np.testing.assert_allclose(srv.wait(k), _plain(env, pop, dom, t), rtol=1e-6)
    info = srv.ticket_info(k)
    say(info, srv.stats())
    assert info["cache_hits"] == 8
    assert srv.stats()["failed"] == 0
    srv.close()


def test_no_room_between_the_rows_it_reads(env):
    """Rows of one grid lie so that none of another fits between them; a request
    that reads them and needs new ones is planned without the reads."""
    tgp, ctx, torch = env
    small, large = tgp.Domain(ctx, (32, 32)), tgp.Domain(ctx, (64, 64))   # rows of 4 and 16 KiB
    ts, tl = (torch.zeros(1, d.cases, dtype=torch.float32, device="cuda:0") for d in (small, large))

    def rows(ids, per=8):
        """`per` trees each that share one costly subtree of both sides."""
        return [f"add(pow(sin(exp(mult(x, y))), cos(add(x, {i}.5))), {0.125 * j + i:.3f})" for i in ids for j in range(per)]

    srv = tgp.Server(ctx, cache_budget_bytes=23 * 4096)

    def serve(run, ids, dom, t):
        pop = pg.population_from_texts(rows(ids))
        k = srv.submit(run, pop, dom, t, tgp.MSE)
        np.testing.assert_allclose(srv.wait(k), _plain(env, pop, dom, t), rtol=1e-6)
        return srv.ticket_info(k)
    # four large rows with a small one before each: holes of 4 KiB once the small ones go
    for i in range(4):
        assert serve(1, [i], small, ts)["cache_new"] == 1
        assert serve(0, [i], large, tl)["cache_new"] == 1
    assert srv.stats()["entries"] == 8 and srv.stats()["evictions"] == 0
    srv.end_run(1)
    info = serve(0, [0, 1, 2, 3, 30, 31, 32, 33], large, tl)   # four rows to read, two or more new ones
    print(info, srv.stats(), flush=True)
    assert info["status"] == 0 and info["cache_hits"] == 0
    assert srv.stats()["failed"] == 0
    srv.close()
