"""A context kept for graphs of several sizes: calls of the largest size that
still uses the arrays of a smaller first call, two-sided and SCC (whose in-side
supports lie behind the status bitmaps)."""
import numpy as np
import pytest

import graphgen as gg
from gpu_common import check_all, say
from test_gpu_scc import check_scc
from test_gpu_two_sided import check_two

pytestmark = pytest.mark.gpu


def capacity(n):
    return (n + n // 8 - n // 128 + 64) // 4 * 4


@pytest.fixture
def ctx():
    import paper_2107_12720_amd as T
    c = T.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("first", [4096, 100_000])
def test_two_sided_up_to_the_capacity(ctx, first):
    check_two(ctx, gg.uniform(first, 2 * first, seed=1), algos=(6,), name="first")
    used = ctx.mem_used()
    for n in (capacity(first) - 3, capacity(first)):
        say(f"  n = {n} in the arrays of {first}")
        check_two(ctx, gg.uniform(n, 2 * n, seed=2), algos=(6,), name="uniform")
        check_two(ctx, gg.core_tail(n, seed=3), algos=(6,), name="core+tail")
        check_all(ctx, gg.core_tail(n, seed=4), algos=(6,), name="one-sided")
    assert ctx.mem_used() == used
    n = capacity(first) + 1
    check_two(ctx, gg.core_tail(n, seed=5), algos=(6,), name="grown")


def test_scc_up_to_the_capacity(ctx):
    first = 20_000
    check_scc(ctx, gg.uniform(first, 2 * first, seed=1))
    check_scc(ctx, gg.uniform(capacity(first), 2 * capacity(first), seed=2))
