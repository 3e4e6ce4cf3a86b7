"""Workloads a user of this framework runs, for timing them and checking their results.

listed() gives the fixed ones, draw(rng) one more of the same ranges, prepare(case, seed) what the
program has in hand before the call, run(state) one pass through the public entry points, work(case)
what a pass cannot do without, and exact(case, seed) the result in 64 bits by plain torch.

Graphs are made on the GPU from the seed: R-MAT (a, b, c, d = .57, .19, .19, .05, labels permuted), a
4-neighbour grid with 5 % of its edges rewired, and uniform random graphs; the last two are symmetric.
"""
import math

import numpy as np
import torch

import paper_1904_02241_amd as gc

DEV = "cuda"
DAMPING = 0.85
A, B, C = 0.57, 0.19, 0.19


def listed():
    return [
        # a small graph, ranked by the plain pull: launches and latency
        {"name": "pagerank_small_plain", "kind": "pagerank", "graph": "rmat", "n": 1000, "degree": 8, "form": "pull",
         "width": 0, "range": 0, "dangling": 0, "iters": 20},
        # the largest ranking: R-MAT 24 over blocks of 2^15, the stream layout (the benchmark's default)
        {"name": "pagerank_rmat24_tocab", "kind": "pagerank", "graph": "rmat", "n": 1 << 24, "degree": 16,
         "form": "tocab_pull", "width": 1 << 15, "range": 1 << 14, "dangling": 0, "iters": 20},
        # the push direction (blocks by destination), ranks of sinks leaking, an odd vertex count
        {"name": "pagerank_push_leak", "kind": "pagerank", "graph": "rmat", "n": 3000017, "degree": 16,
         "form": "tocab_push", "width": 1 << 14, "range": 1 << 12, "dangling": 1, "iters": 20},
        # the block width the method was published with, on a graph without hubs
        {"name": "pagerank_wide_uniform", "kind": "pagerank", "graph": "uniform", "n": 2500009, "degree": 16,
         "form": "tocab_pull", "width": 1 << 18, "range": 1 << 12, "dangling": 0, "iters": 20},
        # ranking until the change is small: an ordinary graph, read back every iteration
        {"name": "converge_rmat", "kind": "converge", "graph": "rmat", "n": 300007, "degree": 16, "form": "tocab_pull",
         "width": 1 << 14, "range": 1 << 12, "dangling": 0, "tol": 1e-6},
        # one sparse product with FP32 values
        {"name": "spmv_values", "kind": "spmv", "graph": "rmat", "n": 1 << 22, "degree": 16, "form": "tocab_pull",
         "width": 1 << 15, "range": 1 << 13, "values": "f32"},
        # breadth-first search of a social-network-like graph: few levels, most arcs in one or two of them
        {"name": "bfs_rmat", "kind": "bfs", "graph": "rmat", "n": 1 << 23, "degree": 16, "form": "tocab_pull",
         "width": 1 << 15, "range": 1 << 13},
        # breadth-first search of a road-like graph: many small levels
        {"name": "bfs_grid", "kind": "bfs", "graph": "grid", "n": 2047 * 1931, "rows": 2047, "form": "tocab_pull",
         "width": 1 << 15, "range": 1 << 13},
        # shortest paths, weights of a byte
        {"name": "sssp_uniform", "kind": "sssp", "graph": "uniform", "n": 2000003, "degree": 8, "form": "tocab_pull",
         "width": 1 << 15, "range": 1 << 13, "weight_max": 255},
        # betweenness from a few sources
        {"name": "bc_rmat", "kind": "bc", "graph": "rmat", "n": 1 << 20, "degree": 16, "form": "pull", "width": 0,
         "range": 0, "sources": 2},
        # a graph as it comes in: transposed, cut into blocks, both read back
        {"name": "build_rmat", "kind": "build", "graph": "rmat", "n": 1500007, "degree": 16, "form": "tocab_pull",
         "width": 1 << 15, "range": 1 << 12, "weight_max": 255},
        # many graphs of uneven size and personalised ranks for 64 seeds in one launch
        {"name": "batch_uneven", "kind": "batch", "graph": "rmat", "n": 200003, "graphs": 8, "degree": 16,
         "width": 1 << 16, "seeds": 64, "iters": 20},
    ]


def draw(rng):
    def between(a, b):  # spread over the logarithm, odd sizes among them
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    def graph(lo, hi):
        kind = rng.choice(("rmat", "rmat", "uniform", "grid"))
        c = {"graph": kind, "n": between(lo, hi)}
        if kind == "grid":
            c["rows"] = max(2, int(math.sqrt(c["n"]) * rng.uniform(0.5, 2.0)))
            c["n"] = c["rows"] * max(2, c["n"] // c["rows"])
        else:
            c["degree"] = rng.choice((4, 8, 16))
        return c

    def blocked(c, widths=(12, 13, 14, 15)):
        c["width"] = 1 << rng.choice(widths)
        while c["n"] > 2048 * c["width"]:
            c["width"] *= 2
        c["range"] = 1 << rng.choice((10, 12, 13, 14))
        return c

    kind = rng.choice(("pagerank", "pagerank", "pagerank", "converge", "spmv", "bfs", "bfs", "sssp", "bc", "build", "batch"))
    if kind == "pagerank":
        form = rng.choice(("pull", "push", "tocab_pull", "tocab_pull", "tocab_wide", "tocab_push"))
        c = graph(600, 1 << 20 if form in ("pull", "push") else 8 << 20)
        if form == "tocab_pull":
            blocked(c)
        elif form == "tocab_wide":
            form = "tocab_pull"
            blocked(c, (16, 17, 18))
        elif form == "tocab_push":
            blocked(c, (12, 13, 14))
        else:
            c["width"] = c["range"] = 0
        c.update(form=form, dangling=rng.choice((0, 0, 1)), iters=rng.choice((10, 20)))
    elif kind == "converge":
        c = blocked(graph(600, 4 << 20))
        c.update(form=rng.choice(("tocab_pull", "tocab_pull", "pull")), dangling=0, tol=1e-6)
    elif kind == "spmv":
        c = blocked(graph(600, 6 << 20), (14, 15, 15, 18))
        c.update(form=rng.choice(("tocab_pull", "tocab_pull", "pull")), values=rng.choice(("f32", "f32", "one")))
    elif kind in ("bfs", "sssp"):
        c = blocked(graph(600, 8 << 20 if kind == "bfs" else 3 << 20), (14, 15, 15, 18))
        c["form"] = rng.choice(("tocab_pull", "tocab_pull", "pull"))
        if kind == "sssp":
            c["weight_max"] = rng.choice((255, 255, 60000))
    elif kind == "bc":
        c = graph(600, 1 << 20)
        c.update(form="pull", width=0, range=0, sources=rng.choice((1, 2, 4)))
    elif kind == "build":
        c = blocked(graph(600, 2 << 20))
        c["form"] = rng.choice(("tocab_pull", "tocab_pull", "tocab_push"))
        c["weight_max"] = rng.choice((0, 255))
    else:
        c = {"graph": "rmat", "n": between(1000, 400000), "graphs": rng.randint(1, 12), "degree": rng.choice((8, 16)),
             "width": 1 << rng.choice((16, 17, 18)), "seeds": rng.choice((8, 64)), "iters": rng.choice((10, 20))}
    return {"kind": kind, **c}


# ---------------------------------------------------------------------------
# inputs

def _rand(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)
    return g


def _csr(n, keys):
    """rowptr and colidx (int32) of the arcs src * n + dst in `keys`: no loops, no duplicates, rows ascending."""
    keys = torch.unique(keys)
    src = keys.div(n, rounding_mode="floor")
    dst = keys - src * n
    keep = src != dst
    src, dst = src[keep], dst[keep]
    rowptr = torch.searchsorted(src, torch.arange(n + 1, device=DEV, dtype=torch.int64)).to(torch.int32)
    return rowptr, dst.to(torch.int32)


def _rmat(n, degree, g):
    scale = max(1, (n - 1).bit_length())
    perm = torch.randperm(n, generator=g, device=DEV)
    parts, left, step = [], n * degree, 1 << 25
    while left > 0:
        e = min(left, step)
        left -= e
        u = torch.zeros(e, dtype=torch.int64, device=DEV)
        v = torch.zeros(e, dtype=torch.int64, device=DEV)
        for _ in range(scale):
            r = torch.rand(e, generator=g, device=DEV)
            u = 2 * u + (r >= A + B)
            v = 2 * v + (((r >= A) & (r < A + B)) | (r >= A + B + C))
        keep = (u < n) & (v < n)
        parts.append(perm[u[keep]] * n + perm[v[keep]])
    return _csr(n, torch.cat(parts))


def _symmetric(n, u, v):
    return _csr(n, torch.cat([u * n + v, v * n + u]))


def _uniform(n, degree, g):
    e = n * degree // 2
    return _symmetric(n, torch.randint(0, n, (e,), generator=g, device=DEV), torch.randint(0, n, (e,), generator=g, device=DEV))


def _grid(rows, cols, g):
    i = torch.arange(rows * cols, device=DEV, dtype=torch.int64)
    right = i[i % cols != cols - 1]
    down = i[: (rows - 1) * cols]
    u = torch.cat([right, down])
    v = torch.cat([right + 1, down + cols])
    moved = torch.rand(u.numel(), generator=g, device=DEV) < 0.05
    v = torch.where(moved, torch.randint(0, rows * cols, (u.numel(),), generator=g, device=DEV), v)
    return _symmetric(rows * cols, u, v)


def _graph(case, g):
    n = case["n"]
    if case["graph"] == "rmat":
        return _rmat(n, case["degree"], g)
    if case["graph"] == "uniform":
        return _uniform(n, case["degree"], g)
    return _grid(case["rows"], n // case["rows"], g)


def _sources(rowptr, count, g):
    """Vertices with an out-arc."""
    deg = rowptr[1:] - rowptr[:-1]
    some = torch.nonzero(deg > 0).reshape(-1)
    return some[torch.randint(0, some.numel(), (count,), generator=g, device=DEV)].tolist()


def _inputs(case, seed):
    """The tensors a case is computed from: on the GPU, from the seed alone."""
    g = _rand(seed)
    kind = case["kind"]
    if kind == "batch":
        sizes = [max(64, int(case["n"] / (1 + k) + 13 * k)) for k in range(case["graphs"])]
        graphs = [_rmat(n, case["degree"], g) for n in sizes]
        ppr = _rmat(max(64, case["n"] // 2), case["degree"], g)
        return {"graphs": graphs, "ppr": ppr, "seeds": _sources(ppr[0], case["seeds"], g),
                "ranks": torch.cat([torch.full((n,), 1.0 / n, dtype=torch.float32, device=DEV) for n in sizes])}
    rowptr, colidx = _graph(case, g)
    d = {"rowptr": rowptr, "colidx": colidx}
    n, m = case["n"], colidx.numel()
    if kind in ("pagerank", "converge"):
        d["ranks"] = torch.full((n,), 1.0 / n, dtype=torch.float32, device=DEV)
    elif kind == "spmv":
        d["x"] = torch.rand(n, generator=g, device=DEV)
        d["values"] = torch.rand(m, generator=g, device=DEV) if case["values"] == "f32" else None
    elif kind in ("sssp", "build") and case["weight_max"]:
        d["weight"] = torch.randint(1, case["weight_max"] + 1, (m,), generator=g, device=DEV, dtype=torch.int32)
    if kind in ("bfs", "sssp", "bc"):
        d["sources"] = _sources(rowptr, case.get("sources", 1), g)
    return d


class State(dict):
    """What a pass needs; its handles are given back with it."""

    def __del__(self):
        for h in reversed(self.get("handles", ())):
            h.free()


def _load(s, d):
    s["g"] = gc.graph_load_csr(d["rowptr"], d["colidx"], d.get("weight"), values=d.get("values"))
    s["handles"].append(s["g"])


def _partition(case, g):
    if case["form"] in ("pull", "push"):
        return None
    return gc.tocab_partition(g, gc.GC_PUSH if case["form"] == "tocab_push" else gc.GC_PULL, case["width"], case["range"])


def prepare(case, seed):
    d = _inputs(case, seed)
    s = State(case=case, handles=[])
    kind = case["kind"]
    if kind == "batch":
        gs = [gc.graph_load_csr(*a) for a in d["graphs"]]
        p = gc.graph_load_csr(*d["ppr"])
        s["handles"] += gs + [p]
        s["b"] = gc.batch_create(gs, [case["width"]] * len(gs), p, d["seeds"])
        s["handles"].append(s["b"])
        s["ranks"] = d["ranks"]
        s["out"] = torch.empty_like(d["ranks"])
        s["ppr"] = torch.empty((p.n, case["seeds"]), dtype=torch.float32, device=DEV)
        return s
    if kind == "build":
        s.update(d)
        # room for as many arcs as the graph may have; what an array does not fill stays zero
        n, m, B = case["n"], _arcs(case), -(-case["n"] // case["width"])
        sizes = {"t_rowptr": n + 1, "t_colidx": m, "blk_rowoff": B + 1, "row_ptr": m + 1, "id_map": m, "col": m,
                 "range_ptr": (-(-n // case["range"]) + 1) * B}
        if case["weight_max"]:
            sizes.update(t_weight=m, weight=m)
        s["out"] = {k: torch.zeros(v, dtype=torch.int32, device=DEV) for k, v in sizes.items()}
        return s
    _load(s, d)
    n = case["n"]
    s["t"] = _partition(case, s["g"])
    if s["t"] is not None:
        s["handles"].append(s["t"])
    if kind in ("pagerank", "converge"):
        s["ranks"], s["out"] = d["ranks"], torch.empty(n, dtype=torch.float32, device=DEV)
    elif kind == "spmv":
        s["x"], s["out"] = d["x"], torch.empty(n, dtype=torch.float32, device=DEV)
    elif kind == "bc":
        s["sources"], s["out"] = np.asarray(d["sources"], np.int32), torch.empty(n, dtype=torch.float64, device=DEV)
    else:
        s["source"], s["out"] = d["sources"][0], torch.empty(n, dtype=torch.int32, device=DEV)
    return s


# ---------------------------------------------------------------------------
# one pass

def _build(s):
    """Load, partition, and both layouts into the caller's buffers."""
    o = s["out"]
    g = gc.graph_load_csr(s["rowptr"], s["colidx"], s.get("weight"))
    t = _partition(s["case"], g)
    gc.graph_export_transpose(g, o["t_rowptr"], o["t_colidx"], o.get("t_weight"))
    gc.tocab_export(t, o["blk_rowoff"], o["row_ptr"], o["id_map"], o["col"], o.get("weight"), o["range_ptr"])
    t.free()
    g.free()
    return o


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "pagerank":
        gc.pagerank_iter(s["g"], s["t"], gc.GC_PUSH if case["form"] == "push" else gc.GC_PULL, DAMPING, case["dangling"],
                         s["ranks"], s["out"], case["iters"])
        return s["out"]
    if kind == "converge":
        iters, _ = gc.pagerank_converge(s["g"], s["t"], gc.GC_PULL, DAMPING, case["dangling"], s["ranks"], s["out"],
                                        case["tol"], 200)
        return {"ranks": s["out"], "iters": iters}
    if kind == "spmv":
        gc.spmv(s["g"], s["t"], s["x"], s["out"])
        return s["out"]
    if kind == "bfs":
        return {"depth": s["out"], "levels": gc.bfs_pull(s["g"], s["t"], s["source"], s["out"], gc.GC_POLICY_HEURISTIC)}
    if kind == "sssp":
        gc.sssp_pull(s["g"], s["t"], s["source"], s["out"], gc.GC_POLICY_HEURISTIC)
        return s["out"]
    if kind == "bc":
        s["out"].zero_()
        gc.bc_accumulate(s["g"], s["t"], s["sources"], s["out"], gc.GC_POLICY_HEURISTIC)
        return s["out"]
    if kind == "build":
        return _build(s)
    gc.batch_run(s["b"], DAMPING, case["iters"], s["ranks"], s["out"], s["ppr"])
    return {"ranks": s["out"], "ppr": s["ppr"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without

def _arcs(case):
    """The arcs of the case's graph, at most (duplicates and loops are dropped)."""
    n = case["n"]
    return 4 * n if case["graph"] == "grid" else n * case["degree"]


def work(case):
    kind, n = case["kind"], case["n"]
    if kind == "batch":
        sizes = [case["n"] / (1 + k) for k in range(case["graphs"])]
        m = sum(sizes) * case["degree"]
        pn = n / 2
        pm = pn * case["degree"]
        per = 4 * m + 12 * sum(sizes) + 4 * pm + 8 * pn * case["seeds"]
        return {"bytes": case["iters"] * per, "flops": case["iters"] * (m + pm * case["seeds"])}
    m = _arcs(case)
    if kind in ("pagerank", "converge"):  # every iteration: each arc's column, the offsets, ranks in and out
        k = case.get("iters", 20)
        return {"bytes": k * (4 * m + 12 * n), "flops": k * (m + 4 * n)}
    if kind == "spmv":  # columns and values, offsets, x and y
        return {"bytes": (8 if case["values"] == "f32" else 4) * m + 12 * n, "flops": 2 * m}
    if kind == "bfs":  # offsets, one arc into every vertex, depths
        return {"bytes": 12 * n, "flops": 0}
    if kind == "sssp":  # every arc with its weight once, offsets, distances
        return {"bytes": 8 * m + 8 * n, "flops": m}
    if kind == "bc":  # every arc forward and backward, path counts, depths, dependencies
        return {"bytes": case["sources"] * (8 * m + 32 * n), "flops": case["sources"] * 3 * m}
    per = 8 if case["weight_max"] else 4  # the arcs in, transposed and blocked
    return {"bytes": 3 * (per * m + 4 * n), "flops": 0}


# ---------------------------------------------------------------------------
# results in 64 bits

def _pagerank64(rowptr, colidx, ranks, dangling, iters=None, tol=None):
    n = rowptr.numel() - 1
    deg = (rowptr[1:] - rowptr[:-1]).to(torch.float64)
    src = torch.repeat_interleave(torch.arange(n, device=DEV, dtype=torch.int32), (rowptr[1:] - rowptr[:-1]).to(torch.int64))
    r = ranks.to(torch.float64)
    sink = deg == 0
    step = 1 << 26
    for _ in range(iters if iters is not None else 200):
        c = torch.where(sink, torch.zeros_like(r), r / deg)
        s = torch.zeros_like(r)
        for a in range(0, colidx.numel(), step):
            s.index_add_(0, colidx[a:a + step], c[src[a:a + step]])
        if not dangling:
            s += r[sink].sum() / n
        new = (1 - float(np.float32(DAMPING))) / n + float(np.float32(DAMPING)) * s
        change = float((new - r).abs().sum())
        r = new
        if tol is not None and change <= tol:
            break
    return r


def _ppr64(rowptr, colidx, seeds, iters):
    n, S = rowptr.numel() - 1, len(seeds)
    deg = (rowptr[1:] - rowptr[:-1]).to(torch.float64)
    src = torch.repeat_interleave(torch.arange(n, device=DEV, dtype=torch.int32), (rowptr[1:] - rowptr[:-1]).to(torch.int64))
    d = float(np.float32(DAMPING))
    p = torch.zeros((n, S), dtype=torch.float64, device=DEV)
    p[torch.tensor(seeds, device=DEV), torch.arange(S, device=DEV)] = 1.0
    sink = deg == 0
    inv = torch.where(sink, torch.zeros_like(deg), 1.0 / deg)
    r = p
    step = 1 << 20
    for _ in range(iters):
        c = r * inv[:, None]
        s = torch.zeros_like(r)
        for a in range(0, colidx.numel(), step):
            s.index_add_(0, colidx[a:a + step], c[src[a:a + step]])
        r = (1 - d) * p + d * (s + r[sink].sum(0)[None, :] * p)
    return r


def _bc64(rowptr, colidx, sources):
    n = rowptr.numel() - 1
    dst = colidx.to(torch.int64)
    src = torch.repeat_interleave(torch.arange(n, device=DEV), (rowptr[1:] - rowptr[:-1]).to(torch.int64))
    bc = torch.zeros(n, dtype=torch.float64, device=DEV)
    for s in sources:
        depth = torch.full((n,), -1, dtype=torch.int32, device=DEV)
        depth[s] = 0
        sigma = torch.zeros(n, dtype=torch.float64, device=DEV)
        sigma[s] = 1.0
        level, arcs = 0, []
        while True:
            on = depth[src] == level
            u, v = src[on], dst[on]
            fresh = depth[v] < 0
            u, v = u[fresh], v[fresh]
            if u.numel() == 0:
                break
            depth[v] = level + 1
            sigma.index_add_(0, v, sigma[u])
            arcs.append((u, v))
            level += 1
        delta = torch.zeros_like(sigma)
        for u, v in reversed(arcs):
            delta.index_add_(0, u, sigma[u] / sigma[v] * (1.0 + delta[v]))
        delta[s] = 0.0
        bc += delta
    return bc


def exact(case, seed):
    kind = case["kind"]
    if kind in ("bfs", "sssp", "build"):
        return None  # whole numbers
    d = _inputs(case, seed)
    if kind == "batch":
        at, ranks = 0, []
        for rowptr, colidx in d["graphs"]:
            n = rowptr.numel() - 1
            ranks.append(_pagerank64(rowptr, colidx, d["ranks"][at:at + n], 0, iters=case["iters"]))
            at += n
        return {"ranks": torch.cat(ranks), "ppr": _ppr64(*d["ppr"], d["seeds"], case["iters"])}
    if kind == "pagerank":
        return _pagerank64(d["rowptr"], d["colidx"], d["ranks"], case["dangling"], iters=case["iters"])
    if kind == "converge":
        return {"ranks": _pagerank64(d["rowptr"], d["colidx"], d["ranks"], case["dangling"], tol=case["tol"]), "iters": None}
    if kind == "spmv":
        n = case["n"]
        deg = (d["rowptr"][1:] - d["rowptr"][:-1]).to(torch.int64)
        x = torch.repeat_interleave(d["x"].to(torch.float64), deg)
        if d["values"] is not None:
            x = x * d["values"].to(torch.float64)
        return torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, d["colidx"], x)
    return _bc64(d["rowptr"], d["colidx"], d["sources"])
