"""Batches with workgroups of every shape of size: graphs near the largest that
keeps its supports in LDS, whose padding depends on the number of lanes."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from gpu_common import say
from test_gpu_small import doubled_path, dying_hub

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2107_12720_amd as T
    c = T.Context(0)
    yield c
    c.close()


@pytest.fixture(scope="module")
def graphs():
    gs = [gg.core_tail(n, seed=n, min_sink=1) for n in (57345, 59904, 59905, 61441, 65536)]
    gs += [doubled_path(900), dying_hub(62000, 1000), gg.core_tail(4096, seed=1, min_sink=1),
           gg.uniform(65000, 130000, seed=3), gg.core_tail(300, seed=2, min_sink=1)]
    want = []
    for g in gs:
        r = oracle.peel(g)
        want.append((oracle.bitmap(r.live), oracle.counts(g, r).T6))
    return gs, want


def pack(graphs):
    vbase = np.cumsum([0] + [g.n for g in graphs]).astype(np.int64)
    ebase = np.cumsum([0] + [g.m for g in graphs]).astype(np.int64)
    row_off = np.concatenate([g.row_off[:-1].astype(np.int64) + e
                              for g, e in zip(graphs, ebase)] + [ebase[-1:]]).astype(np.int32)
    col = np.concatenate([g.col for g in graphs]).astype(np.int32)
    words = np.cumsum([0] + [(g.n + 31) // 32 for g in graphs]).astype(np.int64)
    return vbase, ebase, row_off, col, words


def check_batch(ctx, graphs, want, opts=None):
    import torch
    import paper_2107_12720_amd as T
    vbase, ebase, row_off, col, words = pack(graphs)
    live = torch.full((int(words[-1]),), -1, dtype=torch.int32, device="cuda")
    res = ctx.trim_batch(T.to_device(vbase), T.to_device(row_off), T.to_device(col),
                         T.to_device(words), int(vbase[-1]), int(ebase[-1]), live_bitmaps=live,
                         opts=opts)
    torch.cuda.synchronize()
    got, edges = res.bitmap_numpy(), res.worker_edges.cpu().numpy()
    for i, (g, (bm, t6)) in enumerate(zip(graphs, want)):
        assert np.array_equal(got[words[i]:words[i + 1]], bm), (i, g.n)
        assert edges[i] == t6, (i, g.n)


@pytest.mark.parametrize("block", [192, 320, 768, 832, 960])
def test_supports_near_the_lds_limit(ctx, graphs, block):
    import paper_2107_12720_amd as T
    say(f"  block {block}")
    check_batch(ctx, *graphs, opts=T.make_opts(block=block))
