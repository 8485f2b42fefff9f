"""Memory that only makes the learned order's calls faster: calls that need the
room under a cap get it, and a stream being captured allocates none."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from gpu_common import say

pytestmark = pytest.mark.gpu


def test_spare_memory_goes_when_a_call_needs_the_room():
    import torch
    import paper_2107_12720_amd as T
    from paper_2107_12720_amd import learned
    g = gg.uniform(40_000, 1_700_000, seed=3)
    r = oracle.peel(g)
    dg = T.DeviceGraph.upload(g)
    rev = [T.to_device(x) for x in gg.transpose(g)]
    pbf = T.to_device(learned.to_bf16_bits(learned.init_params(3)).view(np.int16))
    scores = torch.zeros(g.m, dtype=torch.float32, device="cuda")
    want_src = np.repeat(np.arange(g.n), np.diff(g.row_off.astype(np.int64)))
    base = T.Context(0)
    fixed = base.mem_used()
    base.trim_csr(6, g.n, dg.row_off, dg.col)
    one = base.mem_used() - fixed
    base.trim_scc(g.n, dg.row_off, dg.col, *rev)
    scc = base.mem_used() - fixed
    base.close()
    tiles = T.Context(0)
    tiles.order_by_key(dg, scores, 0.0, 1.0, torch.zeros_like(dg.col))
    tile_bytes = tiles.mem_used() - fixed
    tiles.close()
    # what the calls need with the counters of 32 bytes a vertex and 8 of features
    for trim_bytes, call in ((one, "csr"), (scc, "scc")):
        c = T.Context(0, mem_budget=fixed + trim_bytes + tile_bytes + (32 + 8) * g.n)
        for _ in range(2):
            indeg, src = learned.prepare(c, dg)
            c.mlp_score(dg, indeg, src, pbf, scores)
            torch.cuda.synchronize()
            say(f"  {call}: {c.mem_used()} bytes with the spare ones")
            assert np.array_equal(indeg.cpu().numpy(), np.bincount(g.col, minlength=g.n))
            assert np.array_equal(src.cpu().numpy(), want_src)
            if call == "csr":
                res = c.trim_csr(6, g.n, dg.row_off, dg.col)
                torch.cuda.synchronize()
                assert np.array_equal(res.bitmap_numpy()[:(g.n + 31) // 32], oracle.bitmap(r.live))
            else:
                label, st = c.trim_scc(g.n, dg.row_off, dg.col, *rev)
                assert int(torch.unique(label).numel()) == st["n_scc"]
        c.close()


def test_degree_keys_captured_on_a_new_context():
    import torch
    import paper_2107_12720_amd as T
    n, m = 70001, 1 << 25
    gen = torch.Generator(device="cuda").manual_seed(1)
    deg = torch.bincount(torch.randint(0, n, (m,), device="cuda", generator=gen), minlength=n)
    row_off = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    row_off[1:] = deg.cumsum(0).to(torch.int32)
    col = torch.randint(0, n, (m,), device="cuda", generator=gen).to(torch.int32)
    dg = T.DeviceGraph(n, row_off, col)
    want = torch.empty(m, dtype=torch.float32, device="cuda")
    keys = torch.zeros_like(want)
    eager = T.Context(0)
    eager.edge_keys(dg, 0, want)
    for held in (False, True):   # nothing to work in; the table there already
        c = T.Context(0)
        if held:
            c.edge_keys(dg, 0, keys)
        used = c.mem_used()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            c.edge_keys(dg, 0, keys)
        assert c.mem_used() == used
        for _ in range(3):
            keys.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(keys, want)
            eager.edge_keys(dg, 0, want)
            torch.cuda.synchronize()
        del graph
        c.close()
    eager.close()


@pytest.mark.parametrize("n", [1, 4095, 4096, 4097, 70001])
def test_late_registration_of_explicit_graphs_needs_no_round_list(n):
    """Under a cap that holds the plain call's memory, from the size on at which
    the rounds' filters lie in it; the counts as ever."""
    import torch
    import paper_2107_12720_amd as T
    g = gg.core_tail(n, seed=n) if n > 1 else gg.from_edges(1, np.zeros(0, np.int32),
                                                            np.zeros(0, np.int32))
    r = oracle.peel(g)
    dg = T.DeviceGraph.upload(g)
    with T.Context(0) as c:
        c.trim_csr(6, g.n, dg.row_off, dg.col if g.m else None)
        plain = c.mem_used()
    c = T.Context(0, mem_budget=plain if n >= 4096 else 0)
    for _ in range(2):
        res = c.trim_csr(6, g.n, dg.row_off, dg.col if g.m else None,
                         opts=T.make_opts(rounds=4))
        torch.cuda.synchronize()
        assert np.array_equal(res.bitmap_numpy()[:(g.n + 31) // 32], oracle.bitmap(r.live))
        st = res.stats_dict()
        assert (st["edges_total"], st["rounds"], st["rechecks"]) == oracle.counts_deferred(g, r, 4)
    if n >= 4096:
        assert c.mem_used() == plain
    c.close()
