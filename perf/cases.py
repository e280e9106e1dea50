"""Performance cases: what a user of this package asks of it, through its entry points.

Each case is a dict of plain values. `listed()` gives the fixed ones, `draw(rng)`
another one of the same kinds and ranges; `prepare` makes what a program holds
before the call (inputs on the GPU, weights, workspaces), `run` is one pass, and
`exact` recomputes the floating outputs in 64 bits with plain torch.

Graphs are pin-board graphs of the shapes the package is exercised on: pin degree
Zipf(2) clipped, board popularity Zipf(1.5) (or both uniform for the tiny graph),
pin features N(0,1), a board's features the mean of a few of its pins, Glorot-uniform
layers.
"""

import math

import torch

import paper_1806_01973_amd as ps

DEV = "cuda"


# ---- the cases -----------------------------------------------------------------------------
def listed():
    return [
        # The smallest all-node job (2,500 nodes): every kernel is tiny, so launches and
        # dependent latencies are what a user waits for. The layers' default order.
        _embed("embed_tiny_f32", 2000, 500, (64, 64, 64), "f32", "pool_then_dense", 200, 2, 10,
               graph="uniform"),
        # The ordinary all-node job in fp32: 1.2M nodes, 100 walks x 3 hops, top 50.
        _embed("embed_medium_f32", 1_000_000, 200_000, (256, 512, 256), "f32", "dense_then_pool",
               100, 3, 50),
        # The largest: a slice of the single-GPU shard (int64 offsets, bf16, 50 walks x 3 hops).
        _embed("embed_shard_bf16", 8_000_000, 2_000_000, (256, 512, 256), "bf16",
               "dense_then_pool", 50, 3, 50, i64=True),
        # The MapReduce form of the all-node inference (boards pool pins, pins pool boards).
        dict(name="bipartite_medium_f32", kind="bipartite", graph="zipf", pins=1_000_000,
             boards=200_000, d=256, m=512, dout=256, dtype="f32", order="pool_then_dense", T=50),
        # One training minibatch's forward and loss on the 1.2M-node graph.
        _minibatch("minibatch_bf16", 1_000_000, 200_000, (256, 512, 256), "bf16", 2048, 500, 0, 0),
        # One wide layer (visual + text features): 1024 -> 2048 -> 512 in bf16.
        _layer("layer_wide_bf16", 300_000, 60_000, (1024, 2048, 512), "bf16", "dense_then_pool",
               "importance"),
        # One layer as the paper prints it, with the max aggregator, at an odd row count.
        _layer("layer_max_f32", 100_003, 20_011, (256, 512, 256), "f32", "pool_then_dense", "max"),
        # Neighbourhoods of new pins on a live graph: an odd number of sources, longer walks.
        dict(name="neighborhoods_fresh", kind="neighborhoods", graph="zipf", pins=1_000_000,
             boards=200_000, sources=4_099, walks=200, hops=5, T=100),
        # Hard negatives for a training batch, the short and the long walk budget.
        _hardneg("hardneg_4k_walks", 1_000_000, 200_000, 2048, 4096, 4),
        _hardneg("hardneg_32k_walks", 1_000_000, 200_000, 2048, 32768, 4),
        # The output layers over all nodes.
        dict(name="mlp_all_f32", kind="mlp", rows=1_200_000, d=256, hidden=256, dout=256,
             dtype="f32"),
        # A training batch's head: output layers on its targets, then the max-margin loss with
        # shared and hard negatives.
        dict(name="head_bf16", kind="head", pairs=2048, neg=500, hard=4, d=256, hidden=256,
             dout=256, dtype="bf16"),
    ]


def draw(rng):
    kind = rng.choice(["embed", "bipartite", "minibatch", "layer", "neighborhoods", "hardneg",
                       "mlp", "head"])
    dims = rng.choice([(64, 64, 64), (128, 256, 128), (256, 512, 256), (208, 336, 176),
                       (48, 112, 80), (512, 512, 256)])
    dtype = rng.choice(["f32", "bf16"])
    order = rng.choice(["pool_then_dense", "dense_then_pool"])
    walks, hops, T = rng.choice([(100, 3, 50), (50, 3, 50), (200, 2, 10), (33, 4, 27), (64, 2, 64),
                                 (200, 5, 100)])
    graph = rng.choice(["zipf", "zipf", "uniform"])
    if kind == "embed":
        pins = _log(rng, 1_000, 1_000_000)
        c = _embed("", pins, max(8, pins // rng.choice([4, 5, 7])), dims, dtype, order, walks,
                   hops, T, graph=graph, i64=rng.random() < 0.3)
    elif kind == "bipartite":
        pins = _log(rng, 1_000, 1_000_000)
        c = dict(kind=kind, graph=graph, pins=pins, boards=max(8, pins // 5), d=dims[0], m=dims[1],
                 dout=dims[0], dtype=dtype, order=order, T=T)
    elif kind == "minibatch":
        pins = _log(rng, 20_000, 1_000_000)
        c = _minibatch("", pins, pins // 5, dims, dtype, _log(rng, 64, 4096), _log(rng, 32, 512),
                       rng.choice([0, 0, 4]), rng.choice([0, 128, 256]))
    elif kind == "layer":
        dims = rng.choice([dims, dims, (1024, 2048, 512)])
        pool = rng.choice(["importance", "importance", "mean", "max"])
        pins = _log(rng, 1_000, 300_000)
        c = _layer("", pins, max(8, pins // 5), dims, dtype,
                   "pool_then_dense" if pool == "max" else order, pool, rng.choice([10, 50, 64, 100]))
    elif kind == "neighborhoods":
        pins = _log(rng, 10_000, 2_000_000)
        c = dict(kind=kind, graph=graph, pins=pins, boards=pins // 5,
                 sources=_log(rng, 64, 200_000), walks=walks, hops=hops, T=T)
    elif kind == "hardneg":
        pins = _log(rng, 100_000, 1_000_000)
        w = _log(rng, 1024, 32768)
        c = _hardneg("", pins, pins // 5, max(64, min(2048, (1 << 26) // (4 * w))), w, 4)
    elif kind == "mlp":
        c = dict(kind=kind, rows=_log(rng, 500, 1_200_000), d=dims[0], hidden=dims[1],
                 dout=dims[2], dtype=dtype)
    else:
        c = dict(kind=kind, pairs=_log(rng, 64, 4096), neg=_log(rng, 32, 1000),
                 hard=rng.choice([0, 4, 7]), d=dims[0], hidden=dims[1], dout=dims[2], dtype=dtype)
    c.pop("name", None)
    return c


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _embed(name, pins, boards, dims, dtype, order, walks, hops, T, graph="zipf", i64=False):
    return dict(name=name, kind="embed", graph=graph, pins=pins, boards=boards, d=dims[0],
                m=dims[1], dout=dims[2], dtype=dtype, order=order, walks=walks, hops=hops, T=T,
                i64=i64)


def _minibatch(name, pins, boards, dims, dtype, pairs, neg, hard, mlp):
    return dict(name=name, kind="minibatch", graph="zipf", pins=pins, boards=boards, d=dims[0],
                m=dims[1], dout=dims[2], dtype=dtype, order="dense_then_pool", walks=100, hops=3,
                T=50, pairs=pairs, neg=neg, hard=hard, mlp=mlp)


def _layer(name, pins, boards, dims, dtype, order, pool, T=50):
    return dict(name=name, kind="layer", graph="zipf", pins=pins, boards=boards, d=dims[0],
                m=dims[1], dout=dims[2], dtype=dtype, order=order, pool=pool, T=T)


def _hardneg(name, pins, boards, queries, walks, hops):
    return dict(name=name, kind="hardneg", graph="zipf", pins=pins, boards=boards,
                queries=queries, walks=walks, hops=hops, lo=1999, hi=5000, k=4)


# ---- inputs --------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _dt(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _csr(case, seed):
    """(offsets int64, col int32) of the case's pin-board graph."""
    g = _gen(7 * seed + 1)
    P, B = case["pins"], case["boards"]
    cdf = perm = None
    if case["graph"] == "uniform":
        deg = torch.randint(1, 9, (P,), generator=g, device=DEV)
    else:
        k = torch.arange(1, min(500, B) + 1, dtype=torch.float64, device=DEV)
        pmf = torch.cumsum(k.pow(-2.0), 0)
        u = torch.rand(P, generator=g, dtype=torch.float64, device=DEV) * (math.pi ** 2 / 6)
        deg = (torch.searchsorted(pmf, u, right=True) + 1).clamp_(max=len(k))
        cdf = torch.cumsum(torch.arange(1, B + 1, dtype=torch.float64, device=DEV).pow(-1.5), 0)
        perm = torch.randperm(B, generator=g, device=DEV)

    def boards(n):
        if cdf is None:
            return torch.randint(0, B, (n,), generator=g, device=DEV)
        u = torch.rand(n, generator=g, dtype=torch.float64, device=DEV) * cdf[-1]
        return perm[torch.searchsorted(cdf, u, right=True).clamp_(max=B - 1)]

    pin = torch.repeat_interleave(torch.arange(P, device=DEV), deg)
    key = torch.sort(pin * B + boards(len(pin)))[0]
    for _ in range(6):  # a pin's boards are distinct: redraw repeats, then drop what is left
        dup = torch.zeros(len(key), dtype=torch.bool, device=DEV)
        dup[1:] = key[1:] == key[:-1]
        n = int(dup.sum())
        if n == 0:
            break
        key[dup] = key[dup] // B * B + boards(n)
        key = torch.sort(key)[0]
    key = torch.unique_consecutive(key)
    pin, board = key // B, key % B
    back = torch.sort(board * P + pin)[0]
    off = torch.zeros(P + B + 1, dtype=torch.int64, device=DEV)
    deg = torch.cat([torch.bincount(pin, minlength=P), torch.bincount(board, minlength=B)])
    off[1:] = torch.cumsum(deg, 0)
    return off, torch.cat([board + P, back % P]).to(torch.int32)


def _graph(case, csr, table=False):
    off, col = csr
    graph = ps.DeviceGraph(off, col, case["pins"], case["boards"],
                           offsets64=bool(case.get("i64", False)))
    return graph.build_walk_table() if table else graph


def _features(case, seed, csr, boards=True):
    g = _gen(7 * seed + 2)
    P, B, d = case["pins"], case["boards"], case["d"]
    x = torch.empty((P + B if boards else P, d), dtype=_dt(case), device=DEV)
    step = max(1, (1 << 28) // d)
    for r in range(0, P, step):
        r1 = min(P, r + step)
        x[r:r1] = torch.randn((r1 - r, d), generator=g, device=DEV)
    if boards:
        off, col = csr
        for r in range(P, P + B, step):
            r1 = min(P + B, r + step)
            lo, n = off[r:r1], (off[r + 1:r1 + 1] - off[r:r1])
            acc = torch.zeros((r1 - r, d), device=DEV)
            for j in range(4):
                at = (lo + j).clamp_(max=len(col) - 1)
                acc += torch.where((n > j)[:, None], x[(col[at].long()).clamp_(max=P - 1)].float(), 0.0)
            x[r:r1] = acc / n.clamp(1, 4)[:, None]
    return x


def _glorot(g, rows, cols, fan, dt):
    a = math.sqrt(6.0 / fan)
    return ((torch.rand((rows, cols), generator=g, device=DEV) * 2 - 1) * a).to(dt)


def _bias(g, n):
    return (torch.rand(n, generator=g, device=DEV) * 2 - 1) * 0.1


def _layers(case, seed, n):
    g = _gen(7 * seed + 3)
    d, m, out, made = case["d"], case["m"], case["dout"], []
    for _ in range(n):
        made.append(ps.DeviceLayer(_glorot(g, m, d, d + m, _dt(case)), _bias(g, m),
                                   _glorot(g, out, d + m, d + m + out, _dt(case)), _bias(g, out),
                                   dtype=_dt(case), dataflow=case["order"],
                                   pool=case.get("pool", "importance")))
        d = out
    return made


def _mlp(case, seed, d, hidden, out):
    g = _gen(7 * seed + 4)
    return ps.DeviceMLP(_glorot(g, hidden, d, d + hidden, _dt(case)), _bias(g, hidden),
                        _glorot(g, out, hidden, hidden + out, _dt(case)), dtype=_dt(case))


def _unit_rows(g, n, d, dt):
    """Rows as the last layer gives them: not negative, of unit length."""
    z = torch.randn((n, d), generator=g, device=DEV).clamp_(min=0)
    return (z / z.norm(dim=1, keepdim=True).clamp_(min=1e-6)).to(dt)


def _batch(case, seed, csr):
    """Query pins, a positive that shares a board with each, shared and hard negatives."""
    g = _gen(7 * seed + 5)
    off, col = csr
    P, n = case["pins"], case["pairs"]

    def pick(rows):
        u = torch.rand(len(rows), generator=g, dtype=torch.float64, device=DEV)
        deg = off[rows + 1] - off[rows]
        return col[off[rows] + (u * deg).long().clamp_(max=deg.max() - 1).minimum(deg - 1)].long()

    q = torch.randperm(P, generator=g, device=DEV)[:n]
    p = pick(pick(q))
    neg = torch.randint(0, P, (case["neg"],), generator=g, device=DEV)
    hard = torch.randint(0, P, (n, case["hard"]), generator=g, device=DEV)
    return [t.to(torch.int32).contiguous() for t in (q, p, neg, hard)]


def _head_rows(case, seed):
    """h of the batch's targets: queries, positives near them, negatives, hard negatives."""
    g = _gen(7 * seed + 6)
    B, d, dt = case["pairs"], case["d"], _dt(case)
    q = _unit_rows(g, B, d, torch.float32)
    p = (q + 0.7 * _unit_rows(g, B, d, torch.float32)) / 1.4
    h = _unit_rows(g, B * case["hard"], d, torch.float32)
    return torch.cat([q, p, _unit_rows(g, case["neg"], d, torch.float32), h]).to(dt).contiguous()


def prepare(case, seed):
    kind, s = case["kind"], {"case": case, "seed": seed}
    if kind in ("mlp", "head"):
        g = _gen(7 * seed + 6)
        s["mlp"] = _mlp(case, seed, case["d"], case["hidden"], case["dout"])
        s["h"] = (_unit_rows(g, case["rows"], case["d"], _dt(case)) if kind == "mlp"
                  else _head_rows(case, seed))
        return s
    csr = _csr(case, seed)
    if kind == "embed":
        layers = _layers(case, seed, 2)
        s["job"] = ps.EmbedAll(_graph(case, csr), layers, case["walks"], case["hops"], case["T"],
                               seed)
        s["x"] = _features(case, seed, csr)
    elif kind == "bipartite":
        s["job"] = ps.EmbedAllBipartite(_graph(case, csr), _layers(case, seed, 2), case["T"], seed)
        s["x"] = _features(case, seed, csr, boards=False)
    elif kind == "minibatch":
        mlp = _mlp(case, seed, case["dout"], case["mlp"], case["mlp"]) if case["mlp"] else None
        s["job"] = ps.Minibatch(_graph(case, csr, table=True), _layers(case, seed, 2),
                                case["walks"], case["hops"], case["T"], seed, case["pairs"],
                                case["neg"], mlp, case["hard"])
        s["x"] = _features(case, seed, csr)
        s["batch"] = _batch(case, seed, csr)
    elif kind == "layer":
        graph = _graph(case, csr)
        s["layer"] = _layers(case, seed, 1)[0]
        s["nbr"] = ps.build_neighborhoods(graph, 100, 3, case["T"], seed, count_steps=False)[0]
        s["x"] = _features(case, seed, csr)
        n = ps.convolve_workspace_size(s["layer"], case["pins"], s["nbr"].rows)
        s["ws"] = torch.empty(max(1, n), dtype=torch.uint8, device=DEV)
        s["out"] = torch.empty((s["nbr"].rows, case["dout"]), dtype=_dt(case), device=DEV)
    elif kind == "neighborhoods":
        s["graph"] = _graph(case, csr)
        s["sources"] = torch.randint(0, case["pins"], (case["sources"],), generator=_gen(7 * seed + 5),
                                     device=DEV).to(torch.int32)
    else:
        s["graph"] = _graph(case, csr, table=True)
        s["queries"] = torch.randint(0, case["pins"], (case["queries"],), generator=_gen(7 * seed + 5),
                                     device=DEV).to(torch.int32)
    return s


# ---- one pass ------------------------------------------------------------------------------
def _table(nbr):
    return {"idx": nbr.idx, "counts": nbr.counts.view(torch.int16), "weights": nbr.weights}


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind in ("embed", "bipartite"):
        h = s["job"].run(s["x"])
        return {"h": h, "nbr": _table(s["job"].nbr)}
    if kind == "minibatch":
        job, (q, p, neg, hard) = s["job"], s["batch"]
        loss = job.run(s["x"], q, p, neg, 0.1, hard=hard if case["hard"] else None)
        return {"loss": loss, "per_pair": job.per_pair, "z": job.z, "sizes": job.sizes(),
                "steps": job.steps}
    if kind == "layer":
        return ps.convolve_layer(s["layer"], s["x"], case["pins"], s["nbr"], out=s["out"],
                                 workspace=s["ws"])
    if kind == "neighborhoods":
        nbr, steps = ps.build_neighborhoods(s["graph"], case["walks"], case["hops"], case["T"],
                                            s["seed"], sources=s["sources"])
        return {"nbr": _table(nbr), "steps": steps}
    if kind == "hardneg":
        out, steps = ps.hard_negatives(s["graph"], s["queries"], case["k"], s["seed"],
                                       case["walks"], case["hops"], case["lo"], case["hi"],
                                       count_steps=True)
        return {"pins": out, "steps": steps}
    z = ps.output_mlp(s["mlp"], s["h"])
    if kind == "mlp":
        return z
    B, n = case["pairs"], case["neg"]
    hard = z[2 * B + n:].view(B, case["hard"], -1) if case["hard"] else None
    loss, per = ps.max_margin_loss(z[:B], z[B:2 * B], z[2 * B:2 * B + n], 0.1, hard)
    return {"z": z, "loss": loss, "per_pair": per}


# ---- the least work, and how far right answers may lie apart ---------------------------------
def _edges(case):
    per = 4.5 if case["graph"] == "uniform" else 2.5  # about: the mean pin degree
    return per * case["pins"]


def work(case):
    kind = case["kind"]
    es = 4 if case.get("dtype") == "f32" else 2
    if kind in ("mlp", "head"):
        rows = (case["rows"] if kind == "mlp"
                else 2 * case["pairs"] + case["neg"] + case["pairs"] * case["hard"])
        d, hid, out = case["d"], case["hidden"], case["dout"]
        b = es * (rows * (d + out) + hid * (d + out)) + 4 * hid
        f = 2.0 * rows * hid * (d + out)
        if kind == "head":
            f += 2.0 * case["pairs"] * (case["neg"] + case["hard"] + 1) * out
        return {"bytes": b, "flops": f}
    P, N = case["pins"], case["pins"] + case["boards"]
    graph = 4 * (N + 1) + 8 * _edges(case)
    if kind == "neighborhoods":
        return {"bytes": graph + 10 * case["sources"] * case["T"], "flops": 0}
    if kind == "hardneg":
        return {"bytes": graph + 4 * case["queries"] * (1 + case["k"]), "flops": 0}
    d, m, out, T = case["d"], case["m"], case["dout"], case["T"]
    if kind == "minibatch":  # about 40 further pins per target and layer, each row read once
        n1 = min(N, 40 * (2 * case["pairs"] + case["neg"] + case["pairs"] * case["hard"]))
        n0 = min(N, 4 * n1)
        rows = n0 + n1
        return {"bytes": es * n0 * d, "flops": 2.0 * rows * m * (d + out) + 2.0 * n1 * (d + out) * out}
    layers = [(d, m, out), (out, m, out)] if kind != "layer" else [(d, m, out)]
    proj = N if kind == "bipartite" else P
    flops, width = 0.0, 0
    for a, b, c in layers:
        printed = proj * a * b + N * (a + b) * c
        before = proj * b * (a + c) + N * a * c
        flops += 2.0 * (printed if case.get("pool") == "max" else min(printed, before))
        width += 2.0 * N * min(T, 4 if kind == "bipartite" else T) * min(b, c)
    bts = es * ((P if kind == "bipartite" else N) * d + N * out)
    bts += es * sum(b * a + c * (a + b) for a, b, c in layers) + 10 * N * T
    return {"bytes": bts + (graph if kind != "layer" else 0), "flops": flops + width}


def tolerance(case):
    # Visit counts, ids and draws are whole numbers and stay the same. fp32 results move with the
    # order of their sums; bf16 results with the rounding of each stored intermediate.
    if case["kind"] in ("neighborhoods", "hardneg"):
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 2e-4}
    return {"rel": 1e-2, "max": 0.3}


# ---- the same in 64 bits, from the definitions -------------------------------------------------
def _mulhi(a, c):
    return (a * (c >> 16) + ((a * (c & 0xFFFF)) >> 16)) >> 16


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 on int64 tensors holding 32-bit words."""
    M = 0xFFFFFFFF
    k0, k1 = seed & M, (seed >> 32) & M
    c0, c1, c2, c3 = torch.broadcast_tensors(c0, c1, c2, c3)
    for _ in range(10):
        h0, l0 = _mulhi(c0, 0xD2511F53), (c0 * 0xD2511F53) & M
        h1, l1 = _mulhi(c2, 0xCD9E8D57), (c2 * 0xCD9E8D57) & M
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return [c0, c1, c2, c3]


def _word(v):
    return torch.tensor(v, dtype=torch.int64, device=DEV)


def _landings(csr, P, sources, walks, hops, seed):
    """Pins that the walks from each source land on, -1 for none: [sources][walks * hops]."""
    off, col = csr
    n = len(sources)
    u = sources.long()[:, None].expand(n, walks)
    w = torch.arange(walks, device=DEV)[None, :].expand(n, walks)
    cur, landed = u.clone(), torch.zeros((n, walks), dtype=torch.int64, device=DEV)
    land = torch.full((n, walks, hops), -1, dtype=torch.int64, device=DEV)
    active = torch.ones((n, walks), dtype=torch.bool, device=DEV)
    for s in range(2 * hops):
        if s % 4 == 0:
            words = _philox(u, w, _word(s // 4), _word(0), seed)
        lo = off[cur]
        deg = off[cur + 1] - lo
        active = active & (deg > 0)
        at = (lo + ((words[s % 4] * deg) >> 32)).clamp_(max=max(0, len(col) - 1))
        cur = torch.where(active, col[at].long(), cur)
        pin = active & (cur < P)
        old = land.gather(2, landed.clamp(max=hops - 1)[..., None])[..., 0]
        land.scatter_(2, landed.clamp(max=hops - 1)[..., None],
                      torch.where(pin, torch.where(cur != u, cur, -1), old)[..., None])
        landed = landed + pin
        active = active & (landed < hops)
    return land.view(n, walks * hops)


def _top(land, T):
    """Ids (-1: none) and visit counts of the T most visited pins of each row."""
    n, L = land.shape
    v = torch.sort(land, dim=1)[0]
    head = v >= 0
    head[:, 1:] &= v[:, 1:] != v[:, :-1]
    at = torch.arange(L, device=DEV)
    nxt = torch.full((n, L + 1), L, dtype=torch.int64, device=DEV)
    nxt[:, :L] = torch.where(head, at, L)
    nxt = nxt.flip(1).cummin(1)[0].flip(1)[:, 1:]
    big = 1 << 62
    key = torch.where(head, (((1 << 20) - (nxt - at)) << 32) | v, big)
    if L < T:
        key = torch.cat([key, torch.full((n, T - L), big, dtype=torch.int64, device=DEV)], 1)
    key = torch.sort(key, dim=1)[0][:, :T]
    idx = torch.where(key == big, -1, key & 0xFFFFFFFF)
    return idx, torch.where(key == big, 0, (1 << 20) - (key >> 32))


def _neighbors(csr, P, sources, walks, hops, T, seed):
    """(ids int32, weights float64) of the sources' importance neighbourhoods."""
    step = max(1, (3 << 20) // walks)
    idx = torch.empty((len(sources), T), dtype=torch.int32, device=DEV)
    wts = torch.empty((len(sources), T), dtype=torch.float64, device=DEV)
    for r in range(0, len(sources), step):
        i, c = _top(_landings(csr, P, sources[r:r + step], walks, hops, seed), T)
        idx[r:r + step] = i
        wts[r:r + step] = c / c.sum(1, keepdim=True).clamp(min=1)
    return idx, wts


def _convolve(layer, h, n_transform, idx, wts, self_rows=None):
    """One layer in 64 bits; `idx` names rows of the first n_transform rows of h."""
    Q, q, W, w = (t.double() for t in (layer.Q, layer.q, layer.W, layer.w))
    d, dev = layer.d_in, h.device
    linear = layer.pool != "max"
    Wn = W[:, d:].t().contiguous()
    width = layer.d_out if linear else layer.m
    R = torch.empty((n_transform, width), dtype=torch.float64, device=dev)
    for r in range(0, n_transform, 1 << 18):
        p = torch.relu(h[r:min(n_transform, r + (1 << 18))].double() @ Q.t() + q)
        R[r:r + len(p)] = p @ Wn if linear else p
    n = len(idx)
    out = torch.empty((n, layer.d_out), dtype=torch.float64, device=dev)
    step = max(1, (1 << 28) // (width * idx.shape[1]))
    for r in range(0, n, step):
        i = idx[r:r + step].long()
        rows, ok = R[i.clamp(min=0)], i >= 0
        if layer.pool == "max":
            g = rows.masked_fill(~ok[..., None], -math.inf).amax(1)
            g = torch.where(ok.any(1)[:, None], g, 0.0)
        else:
            a = (wts[r:r + step] if layer.pool == "importance"
                 else ok / ok.sum(1, keepdim=True).clamp(min=1))
            g = (rows * torch.where(ok, a, 0.0)[..., None]).sum(1)
        me = h[r:r + len(i)] if self_rows is None else h[self_rows[r:r + len(i)]]
        z = torch.relu(me.double() @ W[:, :d].t() + (g if linear else g @ Wn) + w)
        norm = z.norm(dim=1, keepdim=True)
        out[r:r + step] = torch.where(norm > 0, z / norm, 0.0)
    return out


def _mlp64(mlp, h):
    return torch.cat([torch.relu(x.double() @ mlp.G1.double().t() + mlp.g.double())
                      @ mlp.G2.double().t() for x in h.split(1 << 18)])


def _loss64(zq, zp, zn, zh, margin):
    pos = (zq * zp).sum(1, keepdim=True)
    terms = torch.relu(zq @ zn.t() - pos + margin)
    if zh is not None:
        terms = torch.cat([terms, torch.relu((zq[:, None, :] * zh).sum(2) - pos + margin)], 1)
    per = terms.mean(1)
    return per.mean().reshape(1), per


def exact(case, seed):
    kind = case["kind"]
    if kind == "hardneg":  # whole numbers only
        return None
    if kind in ("mlp", "head"):
        s = prepare(case, seed)
        z = _mlp64(s["mlp"], s["h"])
        if kind == "mlp":
            return z
        # The loss of the head is taken from z as it is stored, as the entry point is given it.
        zs = z.to(_dt(case)).double()
        B, n = case["pairs"], case["neg"]
        hard = zs[2 * B + n:].view(B, case["hard"], -1) if case["hard"] else None
        loss, per = _loss64(zs[:B], zs[B:2 * B], zs[2 * B:2 * B + n], hard, 0.1)
        return {"z": z, "loss": loss, "per_pair": per}
    csr = _csr(case, seed)
    P, N = case["pins"], case["pins"] + case["boards"]
    everyone = torch.arange(N, device=DEV)
    if kind == "neighborhoods":
        src = torch.randint(0, P, (case["sources"],), generator=_gen(7 * seed + 5), device=DEV)
        _, wts = _neighbors(csr, P, src, case["walks"], case["hops"], case["T"], seed)
        return {"nbr": {"idx": None, "counts": None, "weights": wts}, "steps": None}
    if kind == "layer":
        x = _features(case, seed, csr)
        idx, wts = _neighbors(csr, P, everyone, 100, 3, case["T"], seed)
        return _convolve(_layers(case, seed, 1)[0], x, P, idx, wts)
    if kind == "embed":
        idx, wts = _neighbors(csr, P, everyone, case["walks"], case["hops"], case["T"], seed)
        h = _features(case, seed, csr)
        for layer in _layers(case, seed, 2):
            h = _convolve(layer, h, P, idx, wts)
        return {"h": h, "nbr": {"idx": None, "counts": None, "weights": wts}}
    if kind == "bipartite":
        off, col = csr
        T = case["T"]
        lo, deg = off[:-1], off[1:] - off[:-1]
        j = torch.arange(T, device=DEV)
        idx = torch.empty((N, T), dtype=torch.int32, device=DEV)
        for r in range(0, N, 1 << 18):
            b, n = lo[r:r + (1 << 18), None], deg[r:r + (1 << 18), None]
            word = _philox(everyone[r:r + (1 << 18), None], j[None, :], _word(0), _word(2), seed)[0]
            at = b + torch.where(n > T, (word * n) >> 32, j.expand(len(b), T))
            i = col[at.clamp_(max=len(col) - 1)]
            idx[r:r + (1 << 18)] = torch.where((n > T) | (j < n), i, -1)
        # A sampled row's weights are its multiplicities: the mean over its entries with repeats.
        wts = ((idx >= 0) / (idx >= 0).sum(1, keepdim=True).clamp(min=1)).double()
        h = torch.zeros((N, case["d"]), dtype=torch.float64, device=DEV)
        h[:P] = _features(case, seed, csr, boards=False).double()
        for layer in _layers(case, seed, 2):
            h = _convolve(layer, h, N, idx, wts)
        return {"h": h, "nbr": None}
    # minibatch: the sets of the computation graph, then the layers on them.
    q, p, neg, hard = _batch(case, seed, csr)
    ids = torch.cat([q, p, neg, hard.flatten()]).long()
    layers, x = _layers(case, seed, 2), _features(case, seed, csr)
    walk = (case["walks"], case["hops"], case["T"], seed)
    s2 = torch.unique(ids)
    i2, w2 = _neighbors(csr, P, s2, *walk)
    s1 = torch.unique(torch.cat([s2, i2[i2 >= 0].long()]))
    i1, w1 = _neighbors(csr, P, s1, *walk)
    h1 = _convolve(layers[0], x, P, i1, w1, s1)
    local = torch.where(i2 >= 0, torch.searchsorted(s1, i2.long().clamp(min=0)), -1)
    h2 = _convolve(layers[1], h1, len(s1), local, w2, torch.searchsorted(s1, s2))
    if case["mlp"]:
        h2 = _mlp64(_mlp(case, seed, case["dout"], case["mlp"], case["mlp"]), h2)
    z = h2[torch.searchsorted(s2, ids)]
    B, n = case["pairs"], case["neg"]
    zh = z[2 * B + n:].view(B, case["hard"], -1) if case["hard"] else None
    loss, per = _loss64(z[:B], z[B:2 * B], z[2 * B:2 * B + n], zh, 0.1)
    return {"loss": loss, "per_pair": per, "z": z, "sizes": None, "steps": None}
