"""The work a user of the library has it do, as measurable cases.

Each case is a dict of plain values; ``prepare`` makes what a program has in
hand before the call (device graphs, points, a hierarchy, a partition) from a
seed, ``run`` makes one pass through the public entry points of
``paper_0910_2004_amd`` and returns what the path computes, and ``work`` gives
the bytes the path cannot do without (inputs read once, outputs written
once).  Graphs come from the workload families of the package's benchmark:
grids, random geometric graphs of mean degree 8 and R-MAT graphs with
(a, b, c) = (0.57, 0.19, 0.19), generated on the device.

Kinds of case:
  pipeline  validate and coarsen one graph, take the coarsest level, way back
            up with cut and balance per level (one partitioning request)
  batch     many graphs in one union: coarsen together, then every graph's
            hierarchy and way back up
  served    requests admitted to a level-granular server, stepped until all
            have finished
  steps     the method step by step: validate, rate, match, contract, project,
            cut and balance
  relabel   recursive coordinate bisection order and renumbering of a graph
  refined   way back up of a hierarchy with pairwise refinement per level
  refine    pairwise refinement of one level's partition
"""
import math

import numpy as np
import torch

import paper_0910_2004_amd as K

RATINGS = ("expansion*2", "innerOuter", "weight", "expansion", "expansion*")
EPS = (3, 100)


def listed():
    return [
        # the smallest request (a 64 x 64 mesh, bisection): latency and launches
        {"name": "grid_64x64", "kind": "pipeline", "graph": "grid", "rows": 64, "cols": 64,
         "rating": "expansion*2", "k": 2, "wmax": 1},
        # a small served request of odd size, the second rating
        {"name": "rgg_9k_inner_outer", "kind": "pipeline", "graph": "rgg", "n": 9001,
         "rating": "innerOuter", "k": 8, "wmax": 1},
        # the benchmark's geometric graph, both ratings
        {"name": "rgg_1m_expansion_star2", "kind": "pipeline", "graph": "rgg", "n": 1 << 20,
         "rating": "expansion*2", "k": 64, "wmax": 1},
        {"name": "rgg_1m_inner_outer", "kind": "pipeline", "graph": "rgg", "n": 1 << 20,
         "rating": "innerOuter", "k": 64, "wmax": 1},
        # an ordinary power-law request with edge weights
        {"name": "rmat_14_expansion", "kind": "pipeline", "graph": "rmat", "scale": 14,
         "edge_factor": 16, "rating": "expansion", "k": 32, "wmax": 100},
        # the headline workload, the largest graph
        {"name": "rmat_22_expansion_star2", "kind": "pipeline", "graph": "rmat", "scale": 22,
         "edge_factor": 16, "rating": "expansion*2", "k": 256, "wmax": 100},
        # uneven graphs (degraded grids and geometric graphs) in one batch
        {"name": "batch_192", "kind": "batch", "count": 192, "nmin": 1000, "nmax": 64000,
         "rating": "expansion*2", "k": 8, "wmax": 16},
        # the served mix (grids, geometric graphs, R-MAT) on one server
        {"name": "served_24", "kind": "served", "count": 24, "emin": 1000, "emax": 1000000,
         "rating": "innerOuter", "k": 32, "wmax": 1},
        # a program that drives the method step by step
        {"name": "steps_rmat_18", "kind": "steps", "graph": "rmat", "scale": 18, "edge_factor": 16,
         "rating": "expansion*", "k": 64, "wmax": 100},
        # locality renumbering before a partitioning run
        {"name": "rcb_relabel_1m", "kind": "relabel", "n": 1 << 20, "leaf": 32, "wmax": 1},
        # way back up with refinement, and the refinement of one finer level
        {"name": "refined_rgg_64k", "kind": "refined", "graph": "rgg", "n": 1 << 16,
         "rating": "expansion*2", "k": 64, "preset": "fast", "wmax": 1},
        {"name": "refine_rgg_256k", "kind": "refine", "n": (1 << 18) + 1, "k": 16,
         "preset": "fast", "wmax": 1},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, nmax, smax):
    g = rng.choice(("grid", "rgg", "rmat"))
    if g == "grid":
        n = _log_int(rng, 500, nmax)
        rows = max(2, int(round(math.sqrt(n) * rng.uniform(0.5, 2.0))))
        return {"graph": g, "rows": rows, "cols": max(2, n // rows)}
    if g == "rgg":
        return {"graph": g, "n": _log_int(rng, 500, nmax) | 1}
    return {"graph": g, "scale": rng.randint(8, smax), "edge_factor": rng.randint(6, 16)}


def draw(rng):
    kind = rng.choice(("pipeline",) * 5 + ("batch", "served", "steps", "steps", "relabel", "refined",
                                           "refine"))
    c = {"kind": kind, "rating": rng.choice(RATINGS), "wmax": rng.choice((1, 16, 100)),
         "k": rng.choice((2, 8, 32, 64, 256))}
    if kind == "pipeline":
        c.update(_draw_graph(rng, 1 << 20, 21))
        c["k"] = max(k for k in (2, c["k"]) if k == 2 or 40 * k <= _sizes(c)[0])
        if c["graph"] == "rgg" and rng.random() < 0.25:   # the two-phase matcher, in RCB order
            c["block_bits"] = rng.randint(6, 10)
    elif kind == "batch":
        c.update(count=_log_int(rng, 4, 160), nmin=1000, nmax=_log_int(rng, 4000, 64000))
    elif kind == "served":
        c.update(count=_log_int(rng, 2, 20), emin=1000, emax=_log_int(rng, 10000, 800000))
    elif kind == "steps":
        c.update(_draw_graph(rng, 1 << 19, 18))
    elif kind == "relabel":
        c.update(n=_log_int(rng, 1000, 1 << 20) | 1, leaf=rng.choice((1, 8, 32, 500)))
    elif kind == "refined":
        c.update(_draw_graph(rng, 40000, 12))
        c.update(k=rng.choice((2, 8, 32, 64)), preset=rng.choice(("minimal", "fast")))
    else:
        c.update(n=_log_int(rng, 2000, 150000) | 1, k=rng.choice((2, 9, 16, 64)),
                 preset=rng.choice(("minimal", "fast")))
    return c


# ---------------------------------------------------------------------------
# Graphs, generated on the device
# ---------------------------------------------------------------------------
def _csr(n, lo, hi, wmax, gen, cmax=1):
    """Device CSR of the undirected edges {lo, hi} (no loop, no duplicate)."""
    dev = lo.device
    m = lo.numel()
    w = torch.randint(1, wmax + 1, (m,), generator=gen, device=dev, dtype=torch.int32)
    key, order = torch.sort(torch.cat([lo * n + hi, hi * n + lo]))
    ew = torch.cat([w, w])[order]
    adj = (key % n).to(torch.int32)
    xadj = torch.searchsorted(key, torch.arange(n + 1, device=dev, dtype=torch.int64) * n)
    vw = torch.randint(1, cmax + 1, (n,), generator=gen, device=dev, dtype=torch.int32)
    return K.DeviceGraph(n, 2 * m, xadj, adj, ew, vw)


def _grid_edges(rows, cols, gen, drop=0.0):
    idx = torch.arange(rows * cols, device="cuda").reshape(rows, cols)
    lo = torch.cat([idx[:, :-1].reshape(-1), idx[:-1].reshape(-1)])
    hi = torch.cat([idx[:, 1:].reshape(-1), idx[1:].reshape(-1)])
    if drop:
        keep = torch.rand(lo.numel(), generator=gen, device="cuda") >= drop
        lo, hi = lo[keep], hi[keep]
    return lo, hi


def _rgg_edges(pts):
    """Pairs of points closer than sqrt(8 / (pi n)), by cells of that side."""
    n = pts.shape[0]
    r = math.sqrt(8.0 / (math.pi * n))
    m = max(1, int(1.0 / r))
    cell = (pts * m).long().clamp_(max=m - 1)
    cid, at = torch.sort(cell[:, 1] * m + cell[:, 0])
    p = pts[at]
    cx, cy = cell[at, 0], cell[at, 1]
    first = torch.searchsorted(cid, torch.arange(m * m + 1, device=pts.device))
    me = torch.arange(n, device=pts.device)
    los, his = [], []
    for dx, dy in ((0, 0), (1, 0), (-1, 1), (0, 1), (1, 1)):
        x, y = cx + dx, cy + dy
        ok = (x >= 0) & (x < m) & (y < m)
        c = torch.where(ok, y * m + x, 0)
        b, e = first[c], first[c + 1]
        if dx == 0 and dy == 0:
            b = me + 1
        cnt = torch.where(ok, e - b, 0)
        i = torch.repeat_interleave(me, cnt)
        j = torch.arange(i.numel(), device=pts.device) - (torch.cumsum(cnt, 0) - cnt)[i] + b[i]
        near = ((p[i] - p[j]) ** 2).sum(1) < r * r
        u, v = at[i[near]], at[j[near]]
        los.append(torch.minimum(u, v))
        his.append(torch.maximum(u, v))
    return torch.cat(los), torch.cat(his)


def _points(n, gen):
    """n points of the unit square in an order of the seed's.  The point set
    belongs to the size, so that every seed's graph has as many edges (sizes
    of outputs do not change with the seed); the order is the node numbering."""
    fixed = torch.Generator(device="cuda")
    fixed.manual_seed(n)
    pts = torch.rand((n, 2), generator=fixed, device="cuda", dtype=torch.float64)
    return pts[torch.randperm(n, generator=gen, device="cuda")]


def _rmat_edges(scale, edge_factor):
    """The edges belong to the size (weights to the seed), as in _points."""
    n, total = 1 << scale, edge_factor << scale
    gen = torch.Generator(device="cuda")
    gen.manual_seed(total)
    src = torch.zeros(total, dtype=torch.int64, device="cuda")
    dst = torch.zeros(total, dtype=torch.int64, device="cuda")
    for _ in range(scale):
        r = torch.rand(total, generator=gen, device="cuda")
        src = src * 2 + (r >= 0.76)
        dst = dst * 2 + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    keep = src != dst
    src, dst = src[keep], dst[keep]
    key = torch.unique(torch.minimum(src, dst) * n + torch.maximum(src, dst))
    return key // n, key % n


def _graph(c, gen):
    if c["graph"] == "grid":
        return _csr(c["rows"] * c["cols"], *_grid_edges(c["rows"], c["cols"], gen), c["wmax"], gen)
    if c["graph"] == "rgg":
        pts = _points(c["n"], gen)
        g = _csr(c["n"], *_rgg_edges(pts), c["wmax"], gen)
        return K.kappa_relabel(g, K.kappa_rcb_order(pts)) if "block_bits" in c else g
    return _csr(1 << c["scale"], *_rmat_edges(c["scale"], c["edge_factor"]), c["wmax"], gen)


def _sizes(c):
    """(nodes, CSR entries) of a case's graph, expected."""
    if c.get("graph") == "grid":
        r, q = c["rows"], c["cols"]
        return r * q, 2 * (r * (q - 1) + q * (r - 1))
    if c.get("graph") == "rmat":
        return 1 << c["scale"], int(1.9 * (c["edge_factor"] << c["scale"]))
    return c["n"], 8 * c["n"]


def _batch_sizes(c):
    """The batch's graph sizes (the case's own, the same for every seed)."""
    rng = np.random.default_rng(c["count"] * 100003 + c["nmax"])
    return np.rint(np.exp(rng.uniform(math.log(c["nmin"]), math.log(c["nmax"]), c["count"]))).astype(int)


def _served_sizes(c):
    rng = np.random.default_rng(c["count"] * 100003 + c["emax"])
    e = np.exp(rng.uniform(math.log(c["emin"]), math.log(c["emax"]), c["count"]))
    return list(zip(e.tolist(), rng.integers(0, 3, c["count"]).tolist()))


def _union(graphs):
    """The block-diagonal union of device graphs and its node offsets."""
    off = np.zeros(len(graphs) + 1, dtype=np.int64)
    off[1:] = np.cumsum([g.n for g in graphs])
    ent = np.zeros(len(graphs) + 1, dtype=np.int64)
    ent[1:] = np.cumsum([g.nnz for g in graphs])
    xadj = torch.cat([g.xadj[:-1] + int(e) for g, e in zip(graphs, ent)] +
                     [torch.tensor([int(ent[-1])], device="cuda")])
    adj = torch.cat([g.adj + int(o) for g, o in zip(graphs, off)])
    return K.DeviceGraph(int(off[-1]), int(ent[-1]), xadj, adj, torch.cat([g.ew for g in graphs]),
                         torch.cat([g.vw for g in graphs])), off.astype(np.int32)


# ---------------------------------------------------------------------------
def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = {"c": c, "seed": seed}   # also of the tie breaks and of the coarsest partition
    if c["kind"] in ("pipeline", "steps"):
        s["g"] = _graph(c, gen)
        if c["kind"] == "steps":
            s["part"] = torch.randint(0, c["k"], (s["g"].n,), generator=gen, device="cuda",
                                      dtype=torch.int32)
    elif c["kind"] == "batch":
        graphs = []
        for i, n in enumerate(_batch_sizes(c)):
            if i % 2 == 0:
                rows = max(2, int(round(math.sqrt(n))))
                n = rows * max(2, int(round(n / rows)))
                lo, hi = _grid_edges(rows, n // rows, gen, 0.1)
            else:
                lo, hi = _rgg_edges(_points(int(n), gen))
            graphs.append(_csr(int(n), lo, hi, c["wmax"], gen, c["wmax"]))
        s["u"], s["off"] = _union(graphs)
        s["part"] = torch.empty(s["u"].n, dtype=torch.int32, device="cuda")
    elif c["kind"] == "served":
        s["graphs"] = []
        for e, kind in _served_sizes(c):
            if kind == 0:
                side = max(2, int(round(math.sqrt(e / 2))))
                d = {"graph": "grid", "rows": side, "cols": side}
            elif kind == 1:
                d = {"graph": "rgg", "n": max(2, int(round(e / 4)))}
            else:
                d = {"graph": "rmat", "scale": min(20, max(6, int(round(math.log2(e / 16))))),
                     "edge_factor": 16}
            s["graphs"].append(_graph(dict(d, wmax=100 if kind == 2 else c["wmax"]), gen))
        s["off"] = np.cumsum([0] + [g.n for g in s["graphs"]])
        s["part"] = torch.empty(int(s["off"][-1]), dtype=torch.int32, device="cuda")
    elif c["kind"] == "relabel":
        s["xy"] = _points(c["n"], gen)
        s["g"] = _csr(c["n"], *_rgg_edges(s["xy"]), c["wmax"], gen)
    elif c["kind"] == "refined":
        g = _graph(c, gen)
        s["h"] = K.kappa_coarsen(g, K.RATINGS[c["rating"]], seed, 20 * c["k"])
    else:
        # a partition as projected from a coarser level: geometric cells with
        # a frayed border of a few edge lengths
        xy = _points(c["n"], gen)
        s["g"] = _csr(c["n"], *_rgg_edges(xy), c["wmax"], gen)
        side = int(math.isqrt(c["k"]))
        fray = torch.randn((c["n"], 2), generator=gen, device="cuda", dtype=torch.float64)
        at = (xy + fray * (2.0 / math.sqrt(c["n"]))).clamp_(0.0, 1.0 - 1e-9)
        cols = c["k"] // side
        s["part"] = ((at[:, 1] * side).int() * cols + (at[:, 0] * cols).int()).to(torch.int32)
    return s


MAX_LEVELS = 65


def _table(rows):
    """Rows of whole numbers, one per level, in an array of fixed size."""
    out = np.zeros((MAX_LEVELS, len(rows[0])), dtype=np.int64)
    out[:len(rows)] = rows
    return out


def _cuts(results):
    return _table([r.as_tuple() for r in results])


def _coarse_out(coarse, fine):
    """A coarse graph in arrays of the fine graph's size (zeros behind it)."""
    pad, dn, dm = torch.nn.functional.pad, fine.n - coarse.n, fine.nnz - coarse.nnz
    return {"xadj": pad(coarse.xadj, (0, dn)), "adj": pad(coarse.adj, (0, dm)),
            "ew": pad(coarse.ew, (0, dm)), "vw": pad(coarse.vw, (0, dn))}


def _levels(h):
    inf = [h.info(l) for l in range(len(h))]
    return _table([(i.n, i.nnz, i.rounds, i.matched, i.stop_reason) for i in inf])


def run(state):
    s, c = state, state["c"]
    kind = c["kind"]
    if kind == "pipeline":
        h = K.kappa_coarsen(s["g"], K.RATINGS[c["rating"]], s["seed"], 20 * c["k"],
                            block_bits=c.get("block_bits"))
        part, res = K.kappa_uncoarsen(h, c["k"], s["seed"], *EPS)
        return {"part": part, "cuts": _cuts(res), "levels": _levels(h),
                "coarsest": _coarse_out(h.level(len(h) - 1).graph, s["g"])}
    if kind == "batch":
        b = K.kappa_coarsen_batch(s["u"], s["off"], K.RATINGS[c["rating"]], s["seed"], 256)
        off, cuts, info = s["off"], [], []
        for i in range(len(b)):
            h = b.hierarchy(i)
            _, res = K.kappa_uncoarsen(h, c["k"], s["seed"], *EPS,
                                       part0=s["part"][int(off[i]):int(off[i + 1])])
            cuts.append(_cuts(res))
            info.append(b.info(i))
        return {"part": s["part"], "cuts": np.concatenate(cuts), "info": np.array(info)}
    if kind == "served":
        srv = K.Server(K.RATINGS[c["rating"]], s["seed"])
        ids = {srv.admit(g, 20 * c["k"]): i for i, g in enumerate(s["graphs"])}
        cuts = [None] * len(ids)
        while srv.active():
            for rid in srv.step():
                i = ids[rid]
                _, res = K.kappa_uncoarsen(srv.take(rid), c["k"], s["seed"], *EPS,
                                           part0=s["part"][int(s["off"][i]):int(s["off"][i + 1])])
                cuts[i] = _cuts(res)
        return {"part": s["part"], "cuts": np.concatenate(cuts)}
    if kind == "steps":
        g, rating = s["g"], K.RATINGS[c["rating"]]
        status = K.kappa_validate(g)
        num, den = K.kappa_rate(g, rating)
        mate, rounds, matched = K.kappa_match(g, rating, s["seed"])
        cmap, coarse = K.kappa_contract(g, mate)
        cpart = K.kappa_initial_partition(coarse.n, c["k"], 1)
        fine = K.kappa_project(cmap, coarse.n, cpart)
        res, bw = K.kappa_cut_balance(g, fine, c["k"], *EPS)
        res2, bw2 = K.kappa_cut_balance(g, s["part"], c["k"], *EPS)
        return {"status": status, "num": num, "den": den, "mate": mate, "rounds": rounds,
                "matched": matched, "cmap": cmap, "coarse": _coarse_out(coarse, g), "fine": fine,
                "cuts": np.array([res.as_tuple(), res2.as_tuple()]), "bw": bw, "bw2": bw2}
    if kind == "relabel":
        order = K.kappa_rcb_order(s["xy"], c["leaf"])
        g = K.kappa_relabel(s["g"], order)
        return {"order": order, "xadj": g.xadj, "adj": g.adj, "ew": g.ew, "vw": g.vw}
    counts = ("global_iterations", "searches", "moves", "kept", "adoptions", "colours")
    if kind == "refined":
        part, res, st = K.kappa_uncoarsen_refined(s["h"], c["k"], s["seed"], *EPS, preset=c["preset"], seed=3)
        return {"part": part, "cuts": _cuts(res), "stats": _table([[x[q] for q in counts] for x in st])}
    part = s["part"].clone()   # refined in place
    st = K.kappa_refine(s["g"], part, c["k"], *EPS, preset=c["preset"], seed=3)
    return {"part": part, "stats": np.array([st[q] for q in counts])}


def work(case):
    """Inputs read once and outputs written once (ids and weights of 4 bytes,
    offsets of 8); the method has no floating-point work."""
    c = case
    if c["kind"] == "batch":
        n = int(_batch_sizes(c).sum())
        return {"bytes": 12 * n + 8 * 6 * n + 4 * n, "flops": 0}
    if c["kind"] == "served":
        e = sum(x for x, _ in _served_sizes(c))
        return {"bytes": int(16 * e + 16 * e / 6), "flops": 0}
    n, nnz = _sizes(c)
    graph = 12 * n + 8 * nnz
    if c["kind"] == "steps":     # also 16 bytes per rating, mate, cmap, the coarse graph
        return {"bytes": 2 * graph + 16 * nnz + 16 * n, "flops": 0}
    if c["kind"] == "relabel":   # points, order, the graph in and out
        return {"bytes": 20 * n + 2 * graph, "flops": 0}
    if c["kind"] == "refined":   # about twice the finest level in all levels
        return {"bytes": 2 * graph + 4 * n, "flops": 0}
    return {"bytes": graph + 8 * n, "flops": 0}


def exact(case, seed):
    """None: every output is a whole number (ids, counts, weights, exact
    rationals' terms), the same in any correct implementation."""
    return None
