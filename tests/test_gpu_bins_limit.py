"""In-degrees around the edge count from which targets go into several bins."""
import pytest

import graphgen as gg
from test_gpu_prepare import check

pytestmark = pytest.mark.gpu

LIMIT = 11 << 16


@pytest.fixture(scope="module")
def ctx():
    import paper_2107_12720_amd as T
    c = T.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n", [32769, 90_000])
@pytest.mark.parametrize("m", [LIMIT - 1, LIMIT])
def test_limit(ctx, n, m):
    check(ctx, gg.uniform(n, m, seed=m), "uniform")
