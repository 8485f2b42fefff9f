"""AC-6 of large explicit graphs by watched supports (csrc/ac6_watch.h): around
its smallest size, graphs that end in its rounds, in its tail and in the lists,
rounds with few, many and very many removals, unaligned offsets."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from gpu_common import check_all, expected, say

pytestmark = pytest.mark.gpu

MIN_N = 65537
ROUNDS = 64          # rounds before supports are registered


@pytest.fixture(scope="module")
def ctx():
    import paper_2107_12720_amd as T
    c = T.Context(0)
    yield c
    c.close()


def doubled_paths(n, depth, width, seed):
    """`width` paths of `depth` vertices v -> next twice (no forest) into sinks,
    the other vertices on a ring, ids permuted: `width` removals a round."""
    rng = np.random.default_rng(seed)
    perm = rng.permutation(n).astype(np.int32)
    k = depth * width
    i = np.arange(k)
    on = i % depth != depth - 1
    src = np.repeat(i[on], 2)
    ring = np.arange(k, n)
    src = np.r_[src, ring]
    dst = np.r_[np.repeat(i[on] + 1, 2), np.roll(ring, -1)]
    return gg.from_edges(n, perm[src], perm[dst])


def rescued(n, depth, seed):
    """A doubled path whose vertices have a third, live successor every other
    step: hand-backs that find another support."""
    rng = np.random.default_rng(seed)
    i = np.arange(depth - 1)
    src = np.r_[np.repeat(i, 2), np.arange(depth, n), np.arange(depth // 2)]
    dst = np.r_[np.repeat(i + 1, 2), np.roll(np.arange(depth, n), -1),
                rng.integers(depth, n, depth // 2)]
    return gg.from_edges(n, src.astype(np.int32), dst.astype(np.int32))


@pytest.mark.parametrize("n", [61440, 61441, MIN_N - 1, MIN_N, MIN_N + 30, 70016, 131071])
def test_sizes(ctx, n):
    check_all(ctx, gg.uniform(n, n + n // 8, seed=n), algos=(6,), name=f"uniform {n}")
    check_all(ctx, gg.core_tail(n, seed=n), algos=(6,), name=f"core+tail {n}")


@pytest.mark.parametrize("n", [4096, 4097, 30000])
def test_dense(ctx, n):
    """Too many edges for one workgroup."""
    check_all(ctx, gg.uniform(n, (1 << 21) + 1, seed=n), algos=(6,), name=f"uniform {n}")
    # 20 layers, each vertex with successors in later ones
    rng = np.random.default_rng(n)
    deg = (1 << 22) // n
    layer = n // 20
    i = np.repeat(np.arange(n - layer), deg)
    lo = (i // layer + 1) * layer
    g = gg.from_edges(n, i.astype(np.int32), rng.integers(lo, n).astype(np.int32))
    check_all(ctx, g, algos=(6,), name=f"layers {n}")


@pytest.mark.parametrize("depth,width", [(3, 20000), (5, 15000), (ROUNDS // 2, 5000),
                                         (ROUNDS - 1, 600), (ROUNDS, 50), (ROUNDS + 1, 100), (ROUNDS + 2, 700),
                                         (300, 3), (2000, 1)])
def test_depths(ctx, depth, width):
    g = doubled_paths(200003, depth, width, seed=depth)
    check_all(ctx, g, algos=(6,), name=f"{width} paths of {depth}")


@pytest.mark.parametrize("R,n,depth,width", [(2, 200003, 5, 15000), (3, 70016, 40, 100),
                                             (2, (1 << 20) + 5, 6, 30000), (8, 4097, 300, 3),
                                             (64, 80000, 66, 2), (2, 33, 5, 2)])
def test_counted_rounds(ctx, R, n, depth, width):
    """Late registration: the rounds' counts, then the propagation."""
    import torch
    import paper_2107_12720_amd as T
    for g in (doubled_paths(n, depth, width, seed=R), gg.uniform(n, n + n // 4, seed=R)):
        r, c, bm = expected(g)
        total, rounds, re = oracle.counts_deferred(g, r, R)
        ro, col = T.to_device(g.row_off), T.to_device(g.col)
        for flags in (0, T.FLAG_STEPWISE):
            say(f"  R={R} n={n} flags={flags}")
            res = ctx.trim_csr(6, n, ro, col, opts=T.make_opts(rounds=R, flags=flags))
            torch.cuda.synchronize()
            st = res.stats_dict()
            assert np.array_equal(res.bitmap_numpy()[:(n + 31) // 32], bm)
            assert (st["edges_total"], st["rounds"], st["rechecks"]) == (total, rounds, re)


@pytest.mark.parametrize("depth", [40, 500])
def test_rescued(ctx, depth):
    check_all(ctx, rescued(80000, depth, seed=depth), algos=(6,), name=f"rescued {depth}")


@pytest.mark.parametrize("schedule,block", [(1, 64), (2, 1024), (3, 256)])
def test_schedules_and_blocks(ctx, schedule, block):
    import paper_2107_12720_amd as T
    g = gg.rmat(17, 8, seed=4, chain=2000)
    check_all(ctx, g, algos=(6,), opts=T.make_opts(schedule=schedule, block=block), name="rmat")


@pytest.mark.parametrize("offset", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [70000, 70001])
def test_offset_alignment_and_preset(ctx, offset, n):
    import torch
    import paper_2107_12720_amd as T
    g = gg.core_tail(n, seed=9)
    buf = torch.zeros(n + 1 + offset, dtype=torch.int32, device="cuda")
    ro = buf[offset:]
    ro.copy_(torch.from_numpy(g.row_off))
    col = T.to_device(g.col)
    r, c, bm = expected(g)
    res = ctx.trim_csr(6, n, ro, col)
    torch.cuda.synchronize()
    assert np.array_equal(res.bitmap_numpy()[:(n + 31) // 32], bm)
    assert res.stats_dict()["edges_total"] == c.T6
    preset, pbm = gg.sample_vertices(n, 0.8, seed=offset)
    pbm = pbm.copy()
    if n % 32:
        pbm[-1] |= np.uint32(0xFFFFFFFF) << np.uint32(n % 32)   # bits past n are ignored
    rp = oracle.peel(g, preset=preset)
    cp = oracle.counts(g, rp, preset=preset)
    res = ctx.trim_csr_preset(6, n, ro, col, T.to_device(pbm.view(np.int32)))
    torch.cuda.synchronize()
    say(f"  offset {offset} n {n}: {res.stats_dict()}")
    assert np.array_equal(res.bitmap_numpy()[:(n + 31) // 32], oracle.bitmap(rp.live))
    assert int(res.worker_edges.sum()) == cp.T6 == res.stats_dict()["edges_total"]


def test_watchdog(ctx):
    """A budget too small for the tail's barriers stalls the call; the next one
    on the context is right again."""
    import torch
    import paper_2107_12720_amd as T
    g = doubled_paths(100003, 3000, 1, seed=1)
    r, c, bm = expected(g)
    ro, col = T.to_device(g.row_off), T.to_device(g.col)
    ctx.trim_csr(6, g.n, ro, col, opts=T.make_opts(budget=1))
    assert ctx.status() == -6
    res = ctx.trim_csr(6, g.n, ro, col)
    assert ctx.status() == 0
    torch.cuda.synchronize()
    assert np.array_equal(res.bitmap_numpy()[:(g.n + 31) // 32], bm)
