"""SCC searches of many levels: the level counts and labels, with searches that
never pull, that start from an empty frontier and that run one after another."""
import numpy as np
import pytest

import graphgen as gg
from gpu_common import say, upload
from oracle.scc_ref import canonical, scc_labels

pytestmark = pytest.mark.gpu


def check(g, levels=None):
    import torch
    import paper_2107_12720_amd as T
    with T.Context(0) as ctx:
        dev = upload(g, with_reverse=True)
        for _ in range(2):
            label, st = ctx.trim_scc(g.n, *dev)
            torch.cuda.synchronize()
            assert np.array_equal(canonical(label.cpu().numpy()[:g.n].astype(np.int64)),
                                  scc_labels(g))
            if levels is not None:
                assert st["search_levels"] == levels, st
    return st


@pytest.mark.parametrize("n", [3, 100, 1000])
def test_one_cycle(n):
    # both directions meet every vertex once: the pivot's level, n - 1 that take one vertex each
    # way, and none after the last
    g = gg.from_edges(n, np.arange(n, dtype=np.int32), ((np.arange(n) + 1) % n).astype(np.int32))
    check(g, levels=n)


def test_many_cycles():
    rng = np.random.default_rng(1)
    src, dst, at = [], [], 0
    for k in rng.integers(2, 60, 150):
        v = at + np.arange(k)
        src.append(v), dst.append(np.roll(v, -1))
        at += k
    src, dst = np.concatenate(src), np.concatenate(dst)
    perm = rng.permutation(at)
    st = check(gg.from_edges(at, perm[src].astype(np.int32), perm[dst].astype(np.int32)))
    say(f"  levels {st['search_levels']}")
    assert st["n_scc"] == 150


def test_band():
    n = 5000
    rng = np.random.default_rng(2)
    i = np.arange(n)
    src, dst = np.r_[i, i], np.r_[(i + 1) % n, (i + rng.integers(1, 50, n)) % n]
    check(gg.from_edges(n, src.astype(np.int32), dst.astype(np.int32)))
