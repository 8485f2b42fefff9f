"""Deep, narrow graphs: many passes in one workgroup (csrc/watch.h) or many rounds
over the device (csrc/watch_rounds.h) that hand back few vertices, then support
lists, as one graph and in batches, in each form of the supports, against the
oracle."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from gpu_common import check_all, say
from test_gpu_blocks import check_batch

pytestmark = pytest.mark.gpu

PASSES, FINDS, MIN_N = 64, 64, 16384   # hand-over after that many narrow passes, from MIN_N on


@pytest.fixture(scope="module")
def ctx():
    import paper_2107_12720_amd as T
    c = T.Context(0)
    yield c
    c.close()


def deep(n, depth, width, seed, twigs=0):
    """`width` paths into sinks with every edge twice (no forest), one peeling step
    a vertex; every third path vertex has its edges as
    (next, further on, next), so that its scan stops in between; `twigs` vertices
    hang on path vertices by one edge (removed with them, by the lists' S_last) or
    have a live vertex behind it.  The others are a ring, which a part of the path
    vertices' predecessors (other ring vertices) survive on."""
    rng = np.random.default_rng(seed)
    perm = rng.permutation(n).astype(np.int32)
    k = depth * width
    i = np.arange(k)
    pos = i % depth
    adj = [[] for _ in range(n)]
    for v in i[pos != depth - 1]:
        if v % 3 == 0 and pos[v] < depth - 6:
            adj[v] = [v + 1, v + 5, v + 1]
        else:
            adj[v] = [v + 1, v + 1]
    t = np.arange(k, k + twigs)
    ring = np.arange(k + twigs, n)
    for j, v in enumerate(t):
        at = int(rng.integers(0, k))
        adj[v] = [[at], [at, int(rng.choice(ring))], [at, at]][j % 3]
    for j, v in enumerate(ring):
        adj[v] = [int(ring[(j + 1) % len(ring)])]
        if j % 17 == 0:
            adj[v].insert(0, int(rng.integers(0, k)))
    src = np.repeat(np.arange(n), [len(a) for a in adj])
    return gg.from_edges(n, perm[src], perm[np.concatenate([np.asarray(a, np.int64) for a in adj])])


@pytest.mark.parametrize("schedule", [0, 3])
@pytest.mark.parametrize("n,depth,width,twigs", [(MIN_N - 1, 300, 1, 500), (MIN_N, 300, 1, 500),
                                                 (MIN_N + 1, PASSES + 1, 3, 0),
                                                 (30_000, PASSES + 5, FINDS + 40, 4000),
                                                 (30_000, 400, 7, 9000), (61_000, 1000, 2, 20_000)])
def test_one_graph(ctx, n, depth, width, twigs, schedule):
    import paper_2107_12720_amd as T
    g = deep(n, depth, width, n + depth, twigs)
    check_all(ctx, g, algos=(6,), opts=T.make_opts(schedule=schedule), name=f"{width} x {depth}")


def test_fixed_memory(ctx):
    import torch
    import paper_2107_12720_amd as T
    g = deep(40_000, 500, 3, 1, 5000)
    r = oracle.peel(g)
    res = T.trim_csr_noalloc(g.n, T.to_device(g.row_off), T.to_device(g.col))
    torch.cuda.synchronize()
    assert np.array_equal(res.bitmap_numpy()[:(g.n + 31) // 32], oracle.bitmap(r.live))
    assert int(res.worker_edges.sum()) == oracle.counts(g, r).T6


@pytest.mark.parametrize("block,schedule", [(0, 0), (256, 3), (832, 0)])
def test_batch(ctx, block, schedule):
    """One wavefront's graph, supports in LDS (both sides of the limit from which
    lists may follow), in device memory, and graphs that never hand over beside
    them."""
    import paper_2107_12720_amd as T
    gs = [deep(4000, 1500, 1, 1, 900), deep(4096, 700, 3, 2, 500), deep(3900, PASSES + 6, 50, 9, 0),
          deep(MIN_N - 1, 200, 2, 3, 100), deep(MIN_N, 200, 2, 4, 100),
          deep(65_536, 500, 5, 5, 30_000), deep(65_537, 500, 5, 6, 30_000),
          deep(200_000, PASSES + 30, 20, 7, 50_000),
          gg.core_tail(100_000, seed=8), gg.core_tail(2000, seed=9, min_sink=1)]
    want = []
    for g in gs:
        r = oracle.peel(g)
        want.append((oracle.bitmap(r.live), oracle.counts(g, r).T6))
    say(f"  block {block} schedule {schedule}")
    check_batch(ctx, gs, want, opts=T.make_opts(block=block, schedule=schedule))


def test_large_graph_by_lists_from_the_start(ctx):
    gs = [deep((1 << 19) + 5, 300, 4, 3, 1000)]
    r = oracle.peel(gs[0])
    check_batch(ctx, gs, [(oracle.bitmap(r.live), oracle.counts(gs[0], r).T6)])


def test_watchdog_in_the_lists(ctx):
    """A budget that the passes keep and the lists exceed: the call reports it, and
    the next one is right again."""
    import paper_2107_12720_amd as T
    g = deep(40_000, 2000, 1, 5)
    dev = T.to_device(g.row_off), T.to_device(g.col)
    ctx.trim_csr(6, g.n, *dev, opts=T.make_opts(budget=PASSES + 200))
    assert ctx.status() == -6
    check_all(ctx, g, algos=(6,), name="after a stall")


ROUNDS = 8   # narrow rounds of the device-wide tail


@pytest.mark.parametrize("n,width,depths", [(70_001, 1, (3, ROUNDS - 1, ROUNDS, ROUNDS + 1,
                                                         ROUNDS + 2, ROUNDS + 3, 40)),
                                            (300_007, 2, (ROUNDS + 1, ROUNDS + 3, ROUNDS + 5, 60)),
                                            (300_007, 3, (30,)), (1 << 20, 8, (ROUNDS + 6, 30)),
                                            (1 << 20, 9, (30,))])
def test_device_wide_rounds(ctx, n, width, depths):
    """Narrow rounds over the whole device, around their limit, with the first of
    them in launches of their own; one-sided, with late registration and presets."""
    import torch
    import paper_2107_12720_amd as T
    for depth in depths:
        g = deep(n, depth, width, n + depth, 500)
        say(f"  n={n}: {width} x {depth}")
        r, _ = check_all(ctx, g, algos=(6,), name="deep")
        ro, col = T.to_device(g.row_off), T.to_device(g.col)
        res = ctx.trim_csr(6, n, ro, col, opts=T.make_opts(rounds=4))
        torch.cuda.synchronize()
        st = res.stats_dict()
        assert np.array_equal(res.bitmap_numpy()[:(n + 31) // 32], oracle.bitmap(r.live))
        assert (st["edges_total"], st["rounds"], st["rechecks"]) == oracle.counts_deferred(g, r, 4)
        preset, pbm = gg.sample_vertices(n, 0.97, seed=depth)
        rp = oracle.peel(g, preset=preset)
        res = ctx.trim_csr_preset(6, n, ro, col, T.to_device(pbm.view(np.int32)))
        torch.cuda.synchronize()
        assert np.array_equal(res.bitmap_numpy()[:(n + 31) // 32], oracle.bitmap(rp.live))
        assert int(res.worker_edges.sum()) == oracle.counts(g, rp, preset=preset).T6
