"""Reordering of successor lists (csrc/order.hip) at the edges of its tiles of 4,096
edges: lists that begin, end and cross there, lists over several tiles, empty ones,
keys past both ends of the range and not numbers."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TILE = 4096
LEVELS = 16


@pytest.fixture(scope="module")
def ctx():
    import paper_2107_12720_amd as T
    c = T.Context(0)
    yield c
    c.close()


def by_level(row_off, col, key, lo, hi):
    """Every list in order of falling key level, equal levels as they were."""
    with np.errstate(invalid="ignore"):
        x = (np.float32(hi) - key) * np.float32(LEVELS / (hi - lo))
    x = np.where(np.isnan(x), 0, np.clip(x, -1e9, 1e9))   # not a number: level 0
    lev = np.clip(np.trunc(x), 0, LEVELS - 1).astype(np.int64)
    src = np.repeat(np.arange(row_off.size - 1), np.diff(row_off))
    return col[np.lexsort((np.arange(col.size), lev, src))]


@pytest.mark.parametrize("degrees", [
    [TILE], [TILE, TILE], [TILE - 1, 1, TILE], [1, TILE, TILE - 1, 1], [TILE + 1], [3 * TILE + 5],
    [5, 2 * TILE - 5, 7], [TILE - 3, 3 * TILE + 3, 0, 0, 1], [63, 1, 64, 65, 0, 127, 1],
    [2] * (TILE // 2) + [0, 1], [1] * 5000, [64] * 130, [0, 0, 1, 0],
    [10 * TILE + 17, 3, 0, TILE, 5], list(range(200)), [4095, 2, 4095, 1, 4097],
])
@pytest.mark.parametrize("seed", [0, 1])
def test_lists_and_tiles(ctx, degrees, seed):
    import torch
    import paper_2107_12720_amd as T
    rng = np.random.default_rng(seed)
    deg = np.array(degrees)
    row_off = np.r_[0, np.cumsum(deg)].astype(np.int32)
    n, m = deg.size, int(row_off[-1])
    col = rng.integers(0, n, m).astype(np.int32)
    lo, hi = 0.0, 2.0
    key = rng.uniform(-0.25, 2.25, m).astype(np.float32)
    if seed:   # few levels, and keys at and past the ends
        key = rng.choice(np.array([0, 0.125, 1, 2, -np.inf, np.inf, np.nan], np.float32), m)
    dg = T.DeviceGraph(n, T.to_device(row_off), T.to_device(col))
    out = torch.full((m,), -1, dtype=torch.int32, device="cuda")
    ctx.order_by_key(dg, torch.from_numpy(key).cuda(), lo, hi, out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), by_level(row_off, col, key, lo, hi))
