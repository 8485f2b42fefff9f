"""AC-4's first removals (csrc/ac4.hip, ac4_first): predecessor lists around the
lane's and the wavefront's share, and more removals at once than a workgroup
buffers, one- and two-sided and with preset vertices, against the oracle."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from gpu_common import expected, run_csr, say, upload

pytestmark = pytest.mark.gpu

COOP, BATCH, BUF = 16, 8, 2048


@pytest.fixture(scope="module")
def ctx():
    import paper_2107_12720_amd as T
    c = T.Context(0)
    yield c
    c.close()


def sinks_with(lengths, seed):
    """Sink i has lengths[i] predecessors; half of those have it as their only
    successor (removed with it), the others a live ring vertex as well."""
    rng = np.random.default_rng(seed)
    ring = 50
    src, dst = list(range(ring)), [(i + 1) % ring for i in range(ring)]
    nxt = ring + len(lengths)
    for i, k in enumerate(lengths):
        for _ in range(k):
            src.append(nxt)
            dst.append(ring + i)
            if rng.random() < 0.5:
                src.append(nxt)
                dst.append(int(rng.integers(0, ring)))
            src.append(int(rng.integers(0, ring)))   # so that it has a predecessor, too
            dst.append(nxt)
            nxt += 1
    order = np.argsort(np.asarray(src), kind="stable")
    return gg.from_edges(nxt, np.asarray(src, np.int32)[order], np.asarray(dst, np.int32)[order])


LENGTHS = [0, 1, BATCH - 1, BATCH, BATCH + 1, COOP - 1, COOP, COOP + 1, 63, 64, 65,
           64 * BATCH - 1, 64 * BATCH, 64 * BATCH + 1]


@pytest.mark.parametrize("lengths", [LENGTHS, [0] * 500 + LENGTHS * 3, [6 * BUF], [1] * (3 * BUF)],
                         ids=["edges", "many", "one hub", "one each"])
@pytest.mark.parametrize("schedule", [0, 2])
def test_lengths(ctx, lengths, schedule):
    import torch
    import paper_2107_12720_amd as T
    g = sinks_with(lengths, seed=len(lengths))
    opts = T.make_opts(schedule=schedule)
    r, c, bm = expected(g)
    say(f"  n={g.n} m={g.m} dead={g.n - r.n_live}")
    got, edges, st = run_csr(ctx, g, 4, opts=opts)
    assert np.array_equal(got, bm) and edges == c.T4s == st["edges_total"]
    # two-sided: every removed vertex walks both lists once
    ro, col, rro, rc = upload(g, with_reverse=True)
    r2 = oracle.peel2(g)
    res = ctx.trim_csr_two_sided(4, g.n, ro, col, rro, rc, opts=opts)
    torch.cuda.synchronize()
    assert np.array_equal(res.bitmap_numpy()[:(g.n + 31) // 32], oracle.bitmap(r2.live))
    both = np.diff(g.row_off.astype(np.int64)) + np.bincount(g.col, minlength=g.n)
    assert int(res.worker_edges.sum()) == int(both[np.asarray(r2.live) == 0].sum())
    # preset
    preset, pbm = gg.sample_vertices(g.n, 0.7, seed=3)
    rp = oracle.peel(g, preset=preset)
    cp = oracle.counts(g, rp, preset=preset)
    res = ctx.trim_csr_preset(4, g.n, ro, col, T.to_device(pbm.view(np.int32)), rro, rc, opts=opts)
    torch.cuda.synchronize()
    assert np.array_equal(res.bitmap_numpy()[:(g.n + 31) // 32], oracle.bitmap(rp.live))
    assert int(res.worker_edges.sum()) == cp.T4s
