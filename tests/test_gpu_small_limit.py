"""Around the largest graph that one workgroup takes (csrc/small.hip): both sides
of the limit, and sizes between it and what the LDS holds."""
import pytest

import graphgen as gg
from gpu_common import check_all
from test_gpu_small import doubled_path

pytestmark = pytest.mark.gpu

LIMIT = 7 * 8192


@pytest.fixture(scope="module")
def ctx():
    import paper_2107_12720_amd as T
    c = T.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n", [LIMIT - 1, LIMIT, LIMIT + 1, 61_440, 61_441])
def test_limit(ctx, n):
    check_all(ctx, gg.core_tail(n, seed=n), algos=(6,), name="core+tail")
    check_all(ctx, gg.uniform(n, n + n // 8, seed=n), algos=(6,), name="uniform")


def test_deep(ctx):
    for n in (LIMIT, LIMIT + 1):
        g = doubled_path(900)
        check_all(ctx, gg.CSR(n, *pad(g, n)), algos=(6,), name="deep")


def pad(g, n):
    """The graph with n - g.n more vertices, each with a self-loop."""
    import numpy as np
    k = n - g.n
    m = g.m
    return (np.r_[g.row_off, m + 1 + np.arange(k, dtype=np.int32)].astype(np.int32),
            np.r_[g.col, g.n + np.arange(k, dtype=np.int32)].astype(np.int32))
