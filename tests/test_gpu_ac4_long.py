"""AC-4: long lists of vertices removed from the start (csrc/ac4.hip, ac4_long),
around the ends of pieces, hubs with neighbouring ids, pieces longer than a
wavefront's step, on both sides, against the oracle."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from gpu_common import expected, run_csr, say, upload
from test_gpu_ac4_first import sinks_with

pytestmark = pytest.mark.gpu

STEP = 512   # entries of a step; pieces are whole steps


@pytest.fixture(scope="module")
def ctx():
    import paper_2107_12720_amd as T
    c = T.Context(0)
    yield c
    c.close()


def check(ctx, g, opts=None, keep=None):
    import torch
    import paper_2107_12720_amd as T
    r, c, bm = expected(g)
    say(f"  n={g.n} m={g.m} dead={g.n - r.n_live}")
    got, edges, st = run_csr(ctx, g, 4, opts=opts)
    assert np.array_equal(got, bm) and edges == c.T4s == st["edges_total"]
    ro, col, rro, rc = upload(g, with_reverse=True)
    for x, (a, b, ra, rb) in ((g, (ro, col, rro, rc)),
                              (gg.CSR(g.n, *gg.transpose(g)), (rro, rc, ro, col))):
        r2 = oracle.peel2(x)
        res = ctx.trim_csr_two_sided(4, g.n, a, b, ra, rb, opts=opts)
        torch.cuda.synchronize()
        assert np.array_equal(res.bitmap_numpy()[:(g.n + 31) // 32], oracle.bitmap(r2.live))
        both = np.diff(x.row_off.astype(np.int64)) + np.bincount(x.col, minlength=g.n)
        assert int(res.worker_edges.sum()) == int(both[np.asarray(r2.live) == 0].sum())
    if keep is not None:
        preset, pbm = gg.sample_vertices(g.n, keep, seed=3)
        rp = oracle.peel(g, preset=preset)
        res = ctx.trim_csr_preset(4, g.n, ro, col, T.to_device(pbm.view(np.int32)), rro, rc,
                                  opts=opts)
        torch.cuda.synchronize()
        assert np.array_equal(res.bitmap_numpy()[:(g.n + 31) // 32], oracle.bitmap(rp.live))
        assert int(res.worker_edges.sum()) == oracle.counts(g, rp, preset=preset).T4s


@pytest.mark.parametrize("schedule", [0, 2])
@pytest.mark.parametrize("lengths", [[9], [STEP - 1, STEP, STEP + 1], [2 * STEP, 2 * STEP + 1],
                                     [9, 12 * STEP + 63, 17, 3 * STEP - 1] * 5, [40] * 300],
                         ids=["one", "piece", "two pieces", "mixed", "many"])
def test_lengths(ctx, lengths, schedule):
    import paper_2107_12720_amd as T
    check(ctx, sinks_with(lengths, seed=1), T.make_opts(schedule=schedule), keep=0.6)


@pytest.mark.parametrize("keep", [0.1, 0.5, 0.9])
@pytest.mark.parametrize("scale", [12, 16, 17])
def test_hubs_side_by_side(ctx, scale, keep):
    check(ctx, gg.rmat(scale, 16, seed=scale), keep=keep)


@pytest.mark.parametrize("n,m", [(2, 5000), (70, 200_000), (500, 400_000)])
def test_pieces_longer_than_a_step(ctx, n, m):
    """Few vertices, very long lists, all into a few that are preset or sinks."""
    rng = np.random.default_rng(n)
    src = rng.integers(0, max(1, n - 1), m)
    dst = np.where(rng.random(m) < 0.9, n - 1, rng.integers(0, n, m))   # n - 1 is a sink
    check(ctx, gg.from_edges(n, src.astype(np.int32), dst.astype(np.int32)), keep=0.5)
