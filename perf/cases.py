"""The work that users of this library have it do, as cases for measurement.

Every case goes through the package's public entry points: trimming an explicit
graph with each of the three algorithms, with and without late support
registration and vertex sampling; strongly connected components (two-sided
trimming, the forward-backward search and colouring); the implicit graph; a
batch of packed graphs; and the learned successor order (a training step, the
scoring of all edges, the reordering of all successor lists).

Inputs are the repository's own workloads: core+tail graphs, R-MAT graphs
(0.57, 0.19, 0.19, 0.05) with and without a planted chain, the hashed Zipf
graph and batches of small core+tail graphs, drawn on the GPU from the seed.
An R-MAT graph on n vertices, n no power of two, scales the ids of the next
power of two down to [0, n).
"""
import math

import numpy as np
import torch

import paper_2107_12720_amd as T
from paper_2107_12720_amd import learned

ABC = (0.57, 0.19, 0.19)
KEY_RANGE = (0.0, 4.0)   # of log1p(out-degree), as chosen on the training graphs of the benchmark
TRAIN_STEP = 100         # Adam steps behind the weights of a training case


def listed():
    return [
        # a call inside a program's inner loop: a graph of a thousand vertices
        {"name": "csr_1003", "kind": "csr", "graph": "coretail", "n": 1003, "algo": 6},
        # the small benchmark graph: some 30 peeling steps
        {"name": "csr_coretail_65536", "kind": "csr", "graph": "coretail", "n": 65536, "algo": 6},
        # the benchmark's main step: a power-law graph with one deep chain
        {"name": "csr_rmat22_chain", "kind": "csr", "graph": "rmat", "n": 1 << 22, "ef": 16,
         "chain": 100000, "algo": 6},
        # the largest explicit graph, shallow: late support registration
        {"name": "csr_rmat26_rounds4", "kind": "csr", "graph": "rmat", "n": 1 << 26, "ef": 16,
         "algo": 6, "rounds": 4},
        # the counter-based baseline over the transposed graph
        {"name": "csr_rmat24_ac4", "kind": "csr", "graph": "rmat", "n": 1 << 24, "ef": 16,
         "algo": 4},
        # the sweeping baseline in the vertex-sampling sweep, half of the vertices kept
        {"name": "csr_rmat22_ac3_half", "kind": "csr", "graph": "rmat", "n": 1 << 22, "ef": 16,
         "algo": 3, "keep": 0.5},
        # the application: two-sided trimming, search and trimming again
        {"name": "scc_rmat22_chain", "kind": "scc", "graph": "rmat", "n": 1 << 22, "ef": 16,
         "chain": 100000},
        # on-the-fly successors, the largest vertex count
        {"name": "implicit_2_28", "kind": "implicit", "log2n": 28, "s": 2.1, "zero": 0.2},
        # thousands of small and middling graphs in one call
        {"name": "batch_4096", "kind": "batch", "graphs": 4096, "n_min": 100, "n_max": 100000},
        # one training step of the learned order: gradients on every training graph, then Adam
        {"name": "train_16x16384", "kind": "train", "graphs": 16, "n": 1 << 20, "ef": 16,
         "count": 16384},
        # preprocessing and scoring of every edge of the evaluation graph
        {"name": "score_rmat24", "kind": "score", "graph": "rmat", "n": 1 << 24, "ef": 16},
        # keys and reordering of every successor list of the evaluation graph
        {"name": "order_rmat24", "kind": "order", "graph": "rmat", "n": 1 << 24, "ef": 16},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["csr"] * 6 + ["scc", "implicit", "batch", "train", "score", "order"])
    if kind == "csr":
        algo = rng.choice([6, 6, 6, 4, 3])
        if rng.random() < 0.4:
            c = {"kind": kind, "graph": "coretail", "n": _log(rng, 300, 1 << 20), "algo": algo}
        else:
            c = {"kind": kind, "graph": "rmat", "n": _log(rng, 1 << 14, 1 << 25),
                 "ef": rng.randint(4, 16), "algo": algo}
            if algo == 6 and rng.random() < 0.4:
                c["chain"] = _log(rng, 50, c["n"] // 40)
        if algo == 6 and rng.random() < 0.3:
            c["rounds"] = rng.choice([2, 3, 4, 8])
        elif rng.random() < 0.3:
            c["keep"] = round(rng.uniform(0.1, 0.95), 3)
        return c
    if kind == "scc":
        c = {"kind": kind, "graph": "rmat", "n": _log(rng, 1 << 14, 1 << 23),
             "ef": rng.randint(4, 16)}
        if rng.random() < 0.5:
            c["chain"] = _log(rng, 50, c["n"] // 40)
        return c
    if kind == "implicit":
        return {"kind": kind, "log2n": rng.randint(14, 27), "s": round(rng.uniform(1.8, 2.5), 2),
                "zero": round(rng.uniform(0.1, 0.3), 3)}
    if kind == "batch":
        return {"kind": kind, "graphs": _log(rng, 16, 4096), "n_min": 100,
                "n_max": _log(rng, 1000, 100000)}
    if kind == "train":
        return {"kind": kind, "graphs": rng.randint(1, 16), "n": _log(rng, 1 << 14, 1 << 20),
                "ef": rng.randint(4, 16), "count": _log(rng, 1000, 1 << 17)}
    return {"kind": kind, "graph": "rmat", "n": _log(rng, 1 << 14, 1 << 24),
            "ef": rng.randint(4, 16)}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _csr(n, src, dst):
    """Stable CSR: successor order = edge order."""
    s, order = torch.sort(src, stable=True)
    col = dst[order]
    del order
    ids = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    return torch.searchsorted(s, ids, out_int32=True), col


def _sources(n, row_off):
    deg = (row_off[1:] - row_off[:-1]).long()
    return torch.repeat_interleave(torch.arange(n, dtype=torch.int32, device="cuda"), deg)


def _rmat(n, ef, chain, g):
    """ef * n R-MAT edges without self-loops, in generation order; with a chain
    of `chain` vertices, their own edges in place of the drawn ones."""
    scale = max(1, math.ceil(math.log2(n)))
    m, step = int(ef) * n, 1 << 26
    spare = m // 32   # more than the self-loops
    a, ab, abc = ABC[0], ABC[0] + ABC[1], sum(ABC)
    drop = ids = None
    if chain:
        ids = torch.randperm(n, generator=g, device="cuda")[:chain].int()
        drop = torch.zeros(n, dtype=torch.bool, device="cuda")
        drop[ids.long()] = True
    srcs, dsts = [], []
    for lo in range(0, m + spare, step):
        k = min(step, m + spare - lo)
        src = torch.zeros(k, dtype=torch.int32, device="cuda")
        dst = torch.zeros(k, dtype=torch.int32, device="cuda")
        for _ in range(scale):
            r = torch.rand(k, generator=g, device="cuda")
            low = r < ab
            src = src * 2 + ~low
            dst = dst * 2 + torch.where(low, r >= a, r >= abc)
        if n != 1 << scale:
            src = (src.long() * n >> scale).int()
            dst = (dst.long() * n >> scale).int()
        keep = src != dst
        srcs.append(src[keep])
        dsts.append(dst[keep])
    src, dst = torch.cat(srcs)[:m], torch.cat(dsts)[:m]
    del srcs, dsts
    if chain:
        keep = ~drop[src.long()]
        src, dst = torch.cat([src[keep], ids[:-1]]), torch.cat([dst[keep], ids[1:]])
    return _csr(n, src, dst)


def _core_tail_targets(src, first, size, core, g):
    """A target for each edge of vertex `src` (global ids, its graph's vertices
    first .. first + size - 1): uniform in the core for a core vertex, uniform
    among the higher ids for a tail vertex.  Local ids."""
    u = torch.rand(src.numel(), generator=g, device="cuda", dtype=torch.float64)
    v = src - first
    in_core = v < core
    lo = torch.where(in_core, 0, v + 1)
    k = torch.where(in_core, core, size - 1 - v)
    return torch.minimum(lo + (u * k).long(), lo + k - 1), v


def _core_tail(n, g):
    """Out-degree 8 in the core (70 %), Poisson(3) in the tail, 1 % sinks."""
    core, sink = int(0.7 * n), int(0.01 * n)
    deg = torch.poisson(torch.full((n,), 3.0, device="cuda"), generator=g).long()
    deg[:core] = 8
    deg[n - max(sink, 1):] = 0
    src = torch.repeat_interleave(torch.arange(n, device="cuda"), deg)
    dst, v = _core_tail_targets(src, 0, n, core, g)
    keep = dst != v
    return _csr(n, src[keep].int(), dst[keep].int())


def _batch(case, g):
    """Packed core+tail graphs: sizes evenly spread over their logarithm, in
    random order, mean out-degree in [1, 8], tail fraction in [0.1, 0.6], at
    least one sink."""
    G = case["graphs"]
    u = torch.rand((3, G), generator=g, device="cuda", dtype=torch.float64)
    u[0] = (torch.randperm(G, generator=g, device="cuda") + 0.5) / G
    size = torch.exp(math.log(case["n_min"]) +
                     u[0] * math.log(case["n_max"] / case["n_min"])).long()
    vbase = torch.zeros(G + 1, dtype=torch.int64, device="cuda")
    vbase[1:] = torch.cumsum(size, 0)
    core = size - ((0.1 + 0.5 * u[2]) * size).long()
    sink = torch.clamp((0.01 * size).long(), min=1)
    n = int(vbase[-1])
    gid = torch.repeat_interleave(torch.arange(G, device="cuda"), size)
    deg = torch.poisson((1.0 + 7.0 * u[1])[gid].float(), generator=g).long()
    local = torch.arange(n, device="cuda") - vbase[gid]
    deg[local >= (size - sink)[gid]] = 0
    del local
    src = torch.repeat_interleave(torch.arange(n, device="cuda"), deg)
    ge = gid[src]
    dst, v = _core_tail_targets(src, vbase[ge], size[ge], core[ge], g)
    keep = dst != v
    row_off, col = _csr(n, src[keep].int(), dst[keep].int())
    words = torch.zeros(G + 1, dtype=torch.int64, device="cuda")
    words[1:] = torch.cumsum((size + 31) // 32, 0)
    return vbase, row_off, col, words, n


def _explicit(case, g):
    if case["graph"] == "coretail":
        return _core_tail(case["n"], g)
    return _rmat(case["n"], case["ef"], case.get("chain", 0), g)


def _transpose(n, row_off, col):
    return _csr(n, col, _sources(n, row_off))


def _bitmap(flags):
    n = flags.numel()
    f = torch.zeros((n + 31) // 32 * 32, dtype=torch.int64, device="cuda")
    f[:n] = flags
    w = (f.view(-1, 32) << torch.arange(32, device="cuda")).sum(1)
    return torch.where(w >= 1 << 31, w - (1 << 32), w).int()


def _zipf_table(s):
    """Thresholds floor(P(X <= k) * 2^64) of Zipf(s) clamped at 256, as int64 bit patterns."""
    k = np.arange(1, 257, dtype=np.float64)
    cdf = np.cumsum(k ** -s)
    t = cdf / cdf[-1] * 2.0 ** 64
    t = np.array([min(int(x), (1 << 64) - 1) for x in t], dtype=np.uint64)
    return torch.from_numpy(t.view(np.int64)).cuda()


def _outputs(n_words, workers):
    """Output buffers, as a program that calls in a loop keeps them."""
    out = {"live_bitmap": torch.zeros(n_words, dtype=torch.int32, device="cuda"),
           "worker_edges": torch.zeros(workers, dtype=torch.int64, device="cuda"),
           "stats": torch.zeros(T.STATS_WORDS, dtype=torch.int64, device="cuda")}
    # edges_total, n_live, n_dead and rounds; the words after them describe one
    # schedule of the work and differ from call to call, as the split of
    # edges_total over the workers does
    return out, out["stats"][:4]


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    st = {"kind": kind, "ctx": T.Context(0)}
    ctx = st["ctx"]
    if kind == "csr":
        n = case["n"]
        st["algo"], st["n"] = case["algo"], n
        st["row_off"], st["col"] = _explicit(case, g)
        st["rev"] = _transpose(n, st["row_off"], st["col"]) if case["algo"] == 4 else (None, None)
        st["opts"] = T.make_opts(rounds=case.get("rounds", 0))
        st["out"], st["head"] = _outputs((n + 31) // 32, ctx.num_workers(case["algo"]))
        if "keep" in case:
            st["preset"] = _bitmap(torch.rand(n, generator=g, device="cuda") >= case["keep"])
    elif kind == "scc":
        st["n"] = case["n"]
        row_off, col = _explicit(case, g)
        st["graph"] = (row_off, col, *_transpose(case["n"], row_off, col))
        st["label"] = torch.zeros(case["n"], dtype=torch.int32, device="cuda")
    elif kind == "implicit":
        st["args"] = (case["log2n"], seed * 0x9E3779B97F4A7C15 % (1 << 64),
                      int(case["zero"] * 2.0 ** 64), _zipf_table(case["s"]))
        st["out"], st["head"] = _outputs(max(1, (1 << case["log2n"]) // 32), ctx.num_workers(6))
    elif kind == "batch":
        vbase, row_off, col, words, n = _batch(case, g)
        st["args"] = (vbase, row_off, col, words, n, int(col.numel()))
        out, st["head"] = _outputs(int(words[-1]), 1)
        st["out"] = {"live_bitmaps": out["live_bitmap"], "stats": out["stats"], "graph_edges":
                     torch.zeros(case["graphs"], dtype=torch.int64, device="cuda")}
    elif kind == "train":
        st["graphs"] = []
        for _ in range(case["graphs"]):
            row_off, col = _rmat(case["n"], case["ef"], 0, g)
            dg = T.DeviceGraph(case["n"], row_off, col)
            live = ctx.trim_csr(6, dg.n, row_off, col).live_bitmap
            st["graphs"].append((dg, *learned.prepare(ctx, dg), live))
        st["count"] = case["count"]
        tr = st["trainer"] = learned.Trainer(ctx, seed=int(seed))
        # moments as some way into the training
        tr.m1.normal_(0.0, 1e-3, generator=g)
        tr.m2.uniform_(1e-6, 4e-6, generator=g)
        tr.step = TRAIN_STEP
    else:
        row_off, col = _explicit(case, g)
        dg = st["dg"] = T.DeviceGraph(case["n"], row_off, col)
        if kind == "score":
            st["indeg"] = torch.zeros(dg.n, dtype=torch.int32, device="cuda")
            st["src"] = torch.zeros(dg.m, dtype=torch.int32, device="cuda")
            st["scores"] = torch.zeros(dg.m, dtype=torch.float32, device="cuda")
            st["pbf"] = _weights(seed)
    return st


def _weights(seed):
    """BF16 weights of a network with non-zero biases."""
    p = learned.init_params(int(seed))
    p += np.random.default_rng(int(seed)).normal(0.0, 0.05, p.size).astype(np.float32)
    return torch.from_numpy(learned.to_bf16_bits(p).view(np.int16)).cuda()


# --------------------------------------------------------------------- run
def run(st):
    ctx, kind = st["ctx"], st["kind"]
    if kind == "csr":
        if "preset" in st:
            ctx.trim_csr_preset(st["algo"], st["n"], st["row_off"], st["col"], st["preset"],
                                *st["rev"], opts=st["opts"], **st["out"])
        else:
            ctx.trim_csr(st["algo"], st["n"], st["row_off"], st["col"], *st["rev"],
                         opts=st["opts"], **st["out"])
        return {"live": st["out"]["live_bitmap"], "counts": st["head"]}
    if kind == "scc":
        label, s = ctx.trim_scc(st["n"], *st["graph"], label=st["label"])
        return {"label": label, "n_scc": s["n_scc"], "trimmed": s["trimmed"],
                "giant": s["giant"], "paired": s["paired"]}
    if kind == "implicit":
        ctx.trim_implicit(6, *st["args"], **st["out"])
        return {"live": st["out"]["live_bitmap"], "counts": st["head"]}
    if kind == "batch":
        ctx.trim_batch(*st["args"], **st["out"])
        return {"live": st["out"]["live_bitmaps"], "edges": st["out"]["graph_edges"],
                "counts": st["head"]}
    if kind == "train":
        tr = st["trainer"]
        loss = tr.train_step(st["graphs"], st["count"])
        return {"loss": loss, "params": tr.p32, "m": tr.m1, "v": tr.m2,
                "params_bf16": tr.pbf.view(torch.bfloat16)}
    if kind == "score":
        ctx.mlp_prepare(st["dg"], st["indeg"], st["src"])
        ctx.mlp_score(st["dg"], st["indeg"], st["src"], st["pbf"], st["scores"])
        return {"indeg": st["indeg"], "src": st["src"], "scores": st["scores"]}
    return {"col": learned.reference_order(ctx, st["dg"], 0, key_range=KEY_RANGE)}


# -------------------------------------------------------------------- work
MLP_FLOPS = 2 * (8 * 32 + 32 * 32 + 32)   # forward, per edge


def _edges(case):
    return case["n"] * (case["ef"] if case["graph"] == "rmat" else 6.5)


def work(case):
    kind = case["kind"]
    if kind == "csr":
        # offsets, one successor of every vertex, the bitmap; the counters of
        # AC-4 need no successor
        n = case["n"]
        return {"bytes": (4.0 if case["algo"] == 4 else 8.0) * n + n / 8, "flops": 0}
    if kind == "scc":
        # both offset arrays, every edge once, the labels
        return {"bytes": 12.0 * case["n"] + 4.0 * _edges(case), "flops": 0}
    if kind == "implicit":
        # the bitmap; a degree and a successor hashed for every vertex, some 22
        # integer operations each
        n = 1 << case["log2n"]
        return {"bytes": n / 8, "flops": 44.0 * n}
    if kind == "batch":
        n = case["graphs"] * (case["n_max"] - case["n_min"]) / \
            math.log(case["n_max"] / case["n_min"])
        return {"bytes": 8.0 * n + n / 8, "flops": 0}
    if kind == "train":
        k = float(case["graphs"]) * case["count"]
        # per sampled edge: its ids, four offsets, two in-degrees and two status
        # words; forward and twice that backward
        return {"bytes": 40.0 * k + 26.0 * learned.NPARAM, "flops": 3.0 * MLP_FLOPS * k}
    m = _edges(case)
    if kind == "score":
        # offsets, targets; in-degrees, sources and scores written
        return {"bytes": 8.0 * case["n"] + 12.0 * m, "flops": MLP_FLOPS * m}
    # offsets, targets read and written
    return {"bytes": 4.0 * case["n"] + 8.0 * m, "flops": 0}


# ------------------------------------------------------------------- exact
def _mix64(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _split(p):
    p = p.double()
    return (p[:256].view(32, 8), p[256:288], p[288:1312].view(32, 32), p[1312:1344],
            p[1344:1376], p[1376])


def _features(out, inn, e, u, w, row_off, bits):
    """The eight features of edges e = u -> w in FP64."""
    lu, lw, iu, iw = out[u], out[w], inn[u], inn[w]
    h = bits[(e - row_off[u].long()).clamp(max=bits.numel() - 1)]
    f = [lu, iu, lw, iw, lu - lw]
    f += [((h >> b) & 1).double() * 2 - 1 for b in range(3)]
    return torch.stack(f, 1)


def _tables(n, row_off, col):
    deg = (row_off[1:] - row_off[:-1]).double()
    indeg = torch.bincount(col, minlength=n)
    bits = _mix64(np.arange(int(deg.max()) + 1, dtype=np.uint64)) & np.uint64(7)
    return (torch.log1p(deg), torch.log1p(indeg.double()),
            torch.from_numpy(bits.astype(np.int64)).cuda())


def exact(case, seed):
    if case["kind"] == "score":
        st = prepare(case, seed)
        dg = st["dg"]
        src = _sources(dg.n, dg.row_off)
        out, inn, bits = _tables(dg.n, dg.row_off, dg.col)
        W1, b1, W2, b2, w3, b3 = _split(st["pbf"].view(torch.bfloat16))
        scores = torch.empty(dg.m, dtype=torch.float64, device="cuda")
        for lo in range(0, dg.m, 1 << 22):
            hi = min(dg.m, lo + (1 << 22))
            e = torch.arange(lo, hi, device="cuda")
            f = _features(out, inn, e, src[lo:hi].long(), dg.col[lo:hi].long(), dg.row_off, bits)
            h = torch.relu(torch.relu(f @ W1.T + b1) @ W2.T + b2)
            scores[lo:hi] = h @ w3 + b3
        return {"indeg": None, "src": None, "scores": scores}
    if case["kind"] == "train":
        st = prepare(case, seed)
        tr, count = st["trainer"], st["count"]
        p = tr.pbf.view(torch.bfloat16).double().requires_grad_()
        step = tr.step + 1
        total = 0.0
        for gi, (dg, _, src, live) in enumerate(st["graphs"]):
            # the edges that the step samples
            k = np.arange(count, dtype=np.uint64)
            e = _mix64(np.uint64(1000003 + gi) ^ np.uint64(step << 40) ^ k) % np.uint64(dg.m)
            e = torch.from_numpy(e.astype(np.int64)).cuda()
            u, w = src[e].long(), dg.col[e].long()
            out, inn, bits = _tables(dg.n, dg.row_off, dg.col)
            W1, b1, W2, b2, w3, b3 = _split(p)
            f = _features(out, inn, e, u, w, dg.row_off, bits)
            s = torch.relu(torch.relu(f @ W1.T + b1) @ W2.T + b2) @ w3 + b3
            y, on = (((live[x >> 5] >> (x & 31)) & 1).double() for x in (w, u))
            each = torch.nn.functional.binary_cross_entropy_with_logits(s, y, reduction="none")
            total = total + (on * each).sum() / count
        total.backward()
        g = p.grad
        m = 0.9 * tr.m1.double() + 0.1 * g
        v = 0.999 * tr.m2.double() + 0.001 * g * g
        new = tr.p32.double() - tr.lr * (m / (1 - 0.9 ** step)) / \
            (torch.sqrt(v / (1 - 0.999 ** step)) + 1e-8)
        return {"loss": (total.detach() / len(st["graphs"])).reshape(1), "params": new, "m": m,
                "v": v, "params_bf16": new}
    return None   # whole numbers only
