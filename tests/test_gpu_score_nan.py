"""Weights that are not numbers: a hidden unit of NaN counts as inactive in
scoring as in training, whatever the NaN's sign."""
import numpy as np
import pytest

import graphgen as gg

pytestmark = pytest.mark.gpu

NAN = (0x7FC0, 0xFFC0, 0x7F81, 0xFFFF)   # BF16 bits: quiet and signalling, either sign


@pytest.mark.parametrize("words", [3, 1], ids=["two tables", "one table"])
def test_nan_units_are_inactive(words):
    import torch
    import paper_2107_12720_amd as T
    from paper_2107_12720_amd import learned
    g = gg.rmat(12, 8, seed=4)
    dg = T.DeviceGraph.upload(g)
    with T.Context(0) as c:
        learned.prepare(c, dg)
        used = c.mem_used()
    ctx = T.Context(0, mem_budget=used + 4 * words * g.n)
    indeg, src = learned.prepare(ctx, dg)
    p = learned.init_params(seed=2) + np.random.default_rng(3).normal(0, 0.05, 1377).astype(np.float32)
    bits = learned.to_bf16_bits(p)
    off = bits.copy()
    units = {3: NAN[0], 4: NAN[1], 17: NAN[2], 30: NAN[3]}
    for h, x in units.items():
        bits[8 * h:8 * h + 8] = x          # row h of W1
        off[8 * h:8 * h + 8] = 0           # the same unit switched off
        off[256 + h] = 0xBF80              # by a bias of -1
    bits[256 + 9] = NAN[0]                 # a NaN bias
    off[8 * 9:8 * 9 + 8], off[256 + 9] = 0, 0xBF80
    got = []
    for b in (bits, off):
        scores = torch.full((g.m,), -1.0, dtype=torch.float32, device="cuda")
        ctx.mlp_score(dg, indeg, src, T.to_device(b.view(np.int16)), scores)
        torch.cuda.synchronize()
        got.append(scores.cpu().numpy())
    assert ctx.mem_used() == used + 4 * words * g.n
    ctx.close()
    assert np.isfinite(got[1]).all()
    assert np.array_equal(got[0], got[1])
