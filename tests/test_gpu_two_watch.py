"""Two-sided AC-6 by watched supports (csrc/ac6_two_watch.h): around its smallest
size, graphs that end in its rounds and in the lists, on either side, rounds with
few and with many removals."""
import numpy as np
import pytest

import graphgen as gg
from gpu_common import say
from test_gpu_two_sided import check_two

pytestmark = pytest.mark.gpu

ROUNDS = 64          # rounds before supports are registered


@pytest.fixture(scope="module")
def ctx():
    import paper_2107_12720_amd as T
    c = T.Context(0)
    yield c
    c.close()


def paths(n, depth, width, seed, back, fed=True):
    """`width` paths of `depth` vertices v -> next twice (no forest) from a ring
    into sinks (back: from sources into the ring), the other vertices on the
    ring; unfed, the paths' other ends are free too."""
    rng = np.random.default_rng(seed)
    perm = rng.permutation(n).astype(np.int32)
    k = depth * width
    i = np.arange(k)
    on = i % depth != depth - 1
    ring = np.arange(k, n)
    src, dst = np.repeat(i[on], 2), np.repeat(i[on] + 1, 2)
    if fed:
        top = np.arange(0, k, depth)
        src, dst = np.r_[src, rng.integers(k, n, width)], np.r_[dst, top]
    src, dst = np.r_[src, ring], np.r_[dst, np.roll(ring, -1)]
    if back:
        src, dst = dst, src
    return gg.from_edges(n, perm[src], perm[dst])


@pytest.mark.parametrize("n", [4095, 4096, 4127, 65537])
def test_sizes(ctx, n):
    check_two(ctx, gg.uniform(n, n + n // 2, seed=n), algos=(6,), name=f"uniform {n}")
    check_two(ctx, gg.core_tail(n, seed=n), algos=(6,), name=f"core+tail {n}")


@pytest.mark.parametrize("back", [False, True])
@pytest.mark.parametrize("n,depth,width", [(70001, 3, 20000), (70001, ROUNDS // 2, 600),
                                           (70001, ROUNDS - 1, 300), (70001, ROUNDS, 7),
                                           (70001, ROUNDS + 2, 200), (4096, 900, 2),
                                           (300007, 6, 20000)])
def test_depths(ctx, n, depth, width, back):
    for fed in (True, False):
        say(f"  {width} paths of {depth}, back {back}, fed {fed}")
        check_two(ctx, paths(n, depth, width, depth, back, fed), algos=(6,), name="paths")


@pytest.mark.parametrize("schedule,block", [(1, 64), (2, 1024), (3, 256)])
def test_schedules_and_blocks(ctx, schedule, block):
    import paper_2107_12720_amd as T
    g = gg.rmat(15, 8, seed=4, chain=700)
    check_two(ctx, g, algos=(6,), opts=T.make_opts(schedule=schedule, block=block), name="rmat")
