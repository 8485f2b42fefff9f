"""In-degrees and edge sources (trim_mlp_prepare) at the edges of the binned
count's ranges, against numpy's exact counts."""
import numpy as np
import pytest

import graphgen as gg
from gpu_common import say

pytestmark = pytest.mark.gpu

BIN_V = 1 << 15      # vertices of a bin
MIN_M = 1 << 16      # edges from which targets are binned
TILE = 1 << 14       # targets sorted at a time


@pytest.fixture(scope="module")
def ctx():
    import paper_2107_12720_amd as T
    c = T.Context(0)
    yield c
    c.close()


def check(ctx, g, name):
    import torch
    import paper_2107_12720_amd as T
    say(f"  {name}: n={g.n} m={g.m}")
    dg = T.DeviceGraph.upload(g)
    indeg = torch.full((g.n,), -7, dtype=torch.int32, device="cuda")
    src = torch.full((g.m,), -7, dtype=torch.int32, device="cuda")
    for _ in range(2):   # the scratch of the first call is used again
        ctx.mlp_prepare(dg, indeg, src)
    torch.cuda.synchronize()
    assert np.array_equal(indeg.cpu().numpy(), np.bincount(g.col, minlength=g.n)), name
    assert np.array_equal(src.cpu().numpy(),
                          np.repeat(np.arange(g.n), np.diff(g.row_off.astype(np.int64)))), name


def to_few(n, m, seed):
    """Most edges into three hubs of different bins."""
    rng = np.random.default_rng(seed)
    dst = rng.choice(np.array([0, n // 2, n - 1]), size=m)
    pick = rng.random(m) < 0.1
    dst[pick] = rng.integers(0, n, int(pick.sum()))
    return gg.from_edges(n, rng.integers(0, n, m).astype(np.int32), dst.astype(np.int32))


@pytest.mark.parametrize("n,m", [(1, MIN_M), (100, MIN_M - 1), (BIN_V, MIN_M), (BIN_V + 1, MIN_M),
                                 (BIN_V + 1, MIN_M - 1), (2 * BIN_V, 5 * TILE + 1),
                                 (3 * BIN_V + 5, 64 * TILE), (40 * BIN_V, 1030 * TILE + 77)])
def test_sizes(ctx, n, m):
    check(ctx, gg.uniform(n, m, seed=n + m), "uniform")
    if n > 2:
        check(ctx, to_few(n, m, seed=m), "hubs")


@pytest.mark.parametrize("extra", [0, 1])
def test_bin_limit(ctx, extra):
    """The largest vertex count of the binned path and one above it."""
    n = 1024 * BIN_V + extra
    rng = np.random.default_rng(1)
    check(ctx, gg.from_edges(n, rng.integers(0, n, 300000).astype(np.int32),
                             np.r_[rng.integers(0, n, 299999), n - 1].astype(np.int32)), "limit")


def test_memory_cap():
    """No room for the binned targets, but for the counters' copies: the call
    still works."""
    import paper_2107_12720_amd as T
    g = gg.uniform(BIN_V + 8, 3_000_000, seed=5)
    c = T.Context(0, mem_budget=4 << 20)
    try:
        check(c, g, "capped")
        assert c.mem_used() <= 4 << 20
    finally:
        c.close()


@pytest.mark.parametrize("m", [1, 63, 64, 65, 1000, 70001])
def test_score_forms(m):
    """Scoring with the wide and the narrow vertex table agrees to the bit, over
    partial tile pairs and a list longer than the table of hashed positions."""
    import torch
    import paper_2107_12720_amd as T
    from paper_2107_12720_amd import learned
    n = 900
    rng = np.random.default_rng(m)
    s = np.where(rng.random(m) < 0.5, 7, rng.integers(0, n, m)).astype(np.int32)   # one long list
    g = gg.from_edges(n, s, rng.integers(0, n, m).astype(np.int32))
    dg = T.DeviceGraph.upload(g)
    p = learned.init_params(3) + rng.normal(0, 0.05, T.MLP_PARAMS).astype(np.float32)
    pbf = T.to_device(learned.to_bf16_bits(p).view(np.int16))
    wide = T.Context(0)
    used = wide.mem_used()
    narrow = T.Context(0, mem_budget=used + n * 8)   # room for one word per vertex only
    try:
        indeg, src = learned.prepare(wide, dg)
        got = []
        for c in (wide, narrow):
            scores = torch.zeros(g.m, dtype=torch.float32, device="cuda")
            c.mlp_score(dg, indeg, src, pbf, scores)
            torch.cuda.synchronize()
            got.append(scores.cpu().numpy())
        assert narrow.mem_used() == used + n * 4
        assert np.array_equal(got[0], got[1])
    finally:
        wide.close()
        narrow.close()


@pytest.mark.parametrize("n,m", [((1 << 22), 1 << 25), ((1 << 22) - 1, (1 << 25) + 3),
                                 (70001, 1 << 25), (1000, (1 << 25) - 1)])
def test_degree_keys(n, m):
    """The keys of the degree order: from the table of two-byte degrees (many
    edges) and from the offsets, degrees of 65,534 to 65,536 and more included.
    The table's degrees are exact, so the keys are those of the offsets."""
    import torch
    import paper_2107_12720_amd as T
    gen = torch.Generator(device="cuda").manual_seed(n)
    deg = torch.bincount(torch.randint(0, n, (m - 327674,), device="cuda", generator=gen),
                         minlength=n)
    deg[:5] += torch.tensor([65534, 65535, 65536, 131069, 0], device="cuda")
    m = int(deg.sum())
    row_off = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    row_off[1:] = deg.cumsum(0).to(torch.int32)
    col = torch.randint(0, n, (m,), device="cuda", generator=gen).to(torch.int32)
    col[:5000] = torch.arange(5000, device="cuda", dtype=torch.int32) % 5
    ctx = T.Context(0)
    keys = torch.empty(m, dtype=torch.float32, device="cuda")
    ctx.edge_keys(T.DeviceGraph(n, row_off, col), 0, keys)
    torch.cuda.synchronize()
    want = torch.log1p(deg[col.long()].double())
    ctx.close()
    # log1pf is within 2 ulp
    assert float(((keys.double() - want).abs() / want.clamp(min=1.0)).max()) <= 2 ** -22
