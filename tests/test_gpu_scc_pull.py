"""The pull levels of the SCC search: list lengths around the lane's share and
the wavefront's step, with the only reached neighbour last, first or nowhere."""
import numpy as np
import pytest

import graphgen as gg
from gpu_common import say, upload
from oracle.scc_ref import canonical, scc_labels

pytestmark = pytest.mark.gpu


def rings(k, lists, seed):
    """A ring of k vertices (the pivot's component, made heavy by doubled
    edges) and satellites: satellite i has lists[i] predecessors, all but one
    from a second ring that the first does not reach, and an edge back to the
    first ring.  The one from the first ring is first, last or missing."""
    rng = np.random.default_rng(seed)
    ns = len(lists)
    n = 2 * k + ns
    src, dst = [], []
    for _ in range(8):
        src += list(range(k))
        dst += [(i + 1) % k for i in range(k)]
    src += [k + i for i in range(k)]
    dst += [k + (i + 1) % k for i in range(k)]
    for i, (length, where) in enumerate(lists):
        s = 2 * k + i
        pre = [k + int(x) for x in rng.integers(0, k, length)]
        if where == "first":
            pre[0] = 0
        elif where == "last":
            pre[-1] = 0
        src += pre + [s]
        dst += [s] * length + [int(rng.integers(0, k))]
    order = np.argsort(np.asarray(src), kind="stable")
    g = gg.from_edges(n, np.asarray(src, np.int32)[order], np.asarray(dst, np.int32)[order])
    perm = rng.permutation(n).astype(np.int32)   # ids carry no meaning
    so = np.repeat(np.arange(n), np.diff(g.row_off.astype(np.int64)))
    return gg.from_edges(n, perm[so], perm[g.col])


@pytest.mark.parametrize("where", ["first", "last", "nowhere", "mixed"])
def test_list_lengths(where):
    import torch
    import paper_2107_12720_amd as T
    lengths = [1, 2, 3, 4, 5, 31, 32, 33, 36, 63, 64, 65, 95, 96, 97, 128, 160, 161, 1000, 5000]
    kinds = ["first", "last", "nowhere"]
    lists = [(x, kinds[i % 3] if where == "mixed" else where) for i, x in enumerate(lengths * 5)]
    g = rings(700, lists, seed=len(where))
    ctx = T.Context(0)
    try:
        say(f"  {where}: n={g.n} m={g.m}")
        ro, col, rro, rc = upload(g, with_reverse=True)
        label, st = ctx.trim_scc(g.n, ro, col, rro, rc)
        torch.cuda.synchronize()
        assert np.array_equal(canonical(label.cpu().numpy()[:g.n].astype(np.int64)), scc_labels(g))
        assert st["giant"] >= 700 or where == "nowhere", st
    finally:
        ctx.close()
