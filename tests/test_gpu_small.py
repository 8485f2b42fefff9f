"""AC-6 of small graphs in one workgroup (csrc/watch.h, csrc/small.hip): the
edges of its ranges, against the oracle bit for bit and by exact totals."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from gpu_common import check_all, say

pytestmark = pytest.mark.gpu

N_LDS = 65536        # vertices whose statuses and supports fit LDS
M_MAX = 1 << 21      # edges up to which one workgroup is used


@pytest.fixture(scope="module")
def ctx():
    import paper_2107_12720_amd as T
    c = T.Context(0)
    yield c
    c.close()


def doubled_path(n):
    """v -> v + 1 twice: no support is the last successor, so no forest; one
    peeling step per vertex."""
    src = np.repeat(np.arange(n - 1, dtype=np.int32), 2)
    return gg.from_edges(n, src, src + 1)


def dying_hub(n, spare):
    """Every vertex but the last two has the hub (n - 2) first; the hub's only
    successor is the sink n - 1.  `spare` of them have a live second
    successor (a self-loop), the others die with it: all are handed back in one
    phase, more than the list of one phase holds."""
    src = np.repeat(np.arange(n - 2, dtype=np.int32), 2)
    dst = np.full(2 * (n - 2), n - 2, np.int32)
    dst[1:2 * spare:2] = np.arange(spare, dtype=np.int32)
    return gg.from_edges(n, np.r_[src, np.int32(n - 2)], np.r_[dst, np.int32(n - 1)])


def last_link_cycles(n):
    """Paths of single successors into cycles (never settled by the forest
    rounds) beside a path into a sink."""
    k = n // 2
    nxt = np.arange(1, n + 1, dtype=np.int32)
    nxt[k - 1] = k // 2          # first half: a path into a cycle
    return gg.from_edges(n, np.arange(n - 1, dtype=np.int32), nxt[:n - 1])


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 129, 1023, 1024, 1025, 4095, 4097, N_LDS - 1,
                               N_LDS, N_LDS + 1])
def test_sizes(ctx, n):
    check_all(ctx, gg.uniform(n, n + n // 8 + 1, seed=n), name=f"uniform {n}")
    if n > 200:
        check_all(ctx, gg.core_tail(n, seed=n), algos=(6,), name=f"core+tail {n}")


@pytest.mark.parametrize("make,args", [(doubled_path, (3000,)), (dying_hub, (30000, 20000)),
                                       (dying_hub, (9000, 0)), (last_link_cycles, (5000,)),
                                       (last_link_cycles, (65535,))])
def test_shapes(ctx, make, args):
    check_all(ctx, make(*args), algos=(6,), name=f"{make.__name__}{args}")


@pytest.mark.parametrize("extra", [0, 1])
def test_edge_limit(ctx, extra):
    """At the largest edge count of the one-workgroup path and one above it."""
    check_all(ctx, gg.uniform(60000, M_MAX + extra, seed=2), algos=(6,), name=f"m limit + {extra}")


@pytest.mark.parametrize("schedule", [0, 1, 2, 3])
def test_preset_and_schedules(ctx, schedule):
    import torch
    import paper_2107_12720_amd as T
    g = gg.core_tail(20011, seed=6)
    preset, bm = gg.sample_vertices(g.n, 0.8, seed=1)
    r = oracle.peel(g, preset=preset)
    c = oracle.counts(g, r, preset=preset)
    res = ctx.trim_csr_preset(6, g.n, T.to_device(g.row_off), T.to_device(g.col),
                              T.to_device(bm.view(np.int32)), opts=T.make_opts(schedule=schedule))
    torch.cuda.synchronize()
    assert np.array_equal(res.bitmap_numpy()[:(g.n + 31) // 32], oracle.bitmap(r.live))
    assert int(res.worker_edges.sum()) == c.T6 == res.stats_dict()["edges_total"]
    say(f"  preset, schedule {schedule}: {res.stats_dict()}")


@pytest.mark.parametrize("block,workers", [(0, 0), (64, 3), (256, 40)])
def test_batch_sizes(ctx, block, workers):
    """A batch with graphs at the edges of its size classes: one wavefront's,
    a workgroup's with and without supports in LDS, and lists."""
    import torch
    import paper_2107_12720_amd as T
    sizes = [4095, 4096, 4097, 65535, 65536, 65537, (1 << 19) - 1, 1 << 19, (1 << 19) + 1, 1, 64, 65]
    graphs = [gg.core_tail(n, seed=n, min_sink=1) if n > 100 else gg.uniform(n, 2 * n, seed=n)
              for n in sizes]
    graphs += [doubled_path(700), dying_hub(30000, 20000), last_link_cycles(4000),
               gg.uniform(3000, 70000, seed=1)]   # few vertices, too many edges for a wavefront
    vbase = np.cumsum([0] + [g.n for g in graphs]).astype(np.int64)
    ebase = np.cumsum([0] + [g.m for g in graphs]).astype(np.int64)
    row_off = np.concatenate([g.row_off[:-1].astype(np.int64) + e
                              for g, e in zip(graphs, ebase)] + [ebase[-1:]]).astype(np.int32)
    col = np.concatenate([g.col for g in graphs]).astype(np.int32)
    words = np.cumsum([0] + [(g.n + 31) // 32 for g in graphs]).astype(np.int64)
    live = torch.full((int(words[-1]),), -1, dtype=torch.int32, device="cuda")
    res = ctx.trim_batch(T.to_device(vbase), T.to_device(row_off), T.to_device(col),
                         T.to_device(words), int(vbase[-1]), int(ebase[-1]), live_bitmaps=live,
                         opts=T.make_opts(block=block, workers=workers))
    torch.cuda.synchronize()
    got, edges = res.bitmap_numpy(), res.worker_edges.cpu().numpy()
    for i, g in enumerate(graphs):
        r = oracle.peel(g)
        assert np.array_equal(got[words[i]:words[i + 1]], oracle.bitmap(r.live)), (i, g.n)
        assert edges[i] == oracle.counts(g, r).T6, (i, g.n)
