"""GPU parity of the construction steps: transpose (graph_load_csr) and the
TOCAB partition, both bit-exact against the oracle."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from tests import graphs
from tests.gpu_util import load

pytestmark = pytest.mark.gpu

GRAPHS = {
    "rmat16": lambda: gg.rmat(16, 16, seed=1),
    "rmat17_noperm": lambda: gg.rmat(17, 16, seed=2, permute=False),  # hub rows > 4096 arcs
    "grid300x301": lambda: gg.grid(300, 301, 0.05, seed=3),
    "uniform": lambda: gg.uniform(70001, 200000, seed=4),
    "dangling_mix": graphs.dangling_mix,
    "star_in": lambda: graphs.star_in(9000),  # one in-row of 8999 arcs
    "edgeless": lambda: graphs.edgeless(5),
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_transpose_bit_exact(name):
    import paper_1904_02241_amd as gc
    g = GRAPHS[name]().with_weights(7)
    print(f"transpose {name} n={g.n} m={g.m}", flush=True)
    h = load(g, weights=True)
    tr = np.empty(g.n + 1, np.int32)
    tc = np.empty(max(g.m, 1), np.int32)
    tw = np.empty(max(g.m, 1), np.int32)
    gc.graph_export_transpose(h, tr, tc[:g.m] if g.m else tc, tw[:g.m] if g.m else tw)
    gc.gc_sync()
    h.free()
    wr, wc, ww = oracle.transpose(g.n, g.rowptr, g.colidx, g.weights)
    np.testing.assert_array_equal(tr, wr)
    np.testing.assert_array_equal(tc[:g.m], wc)
    np.testing.assert_array_equal(tw[:g.m], ww)


def export_partition(part, g):
    import paper_1904_02241_amd as gc
    info = part.info
    B, P, k = info["B"], info["P"], info["k"]
    R = -(-g.n // k)
    out = dict(blk_rowoff=np.empty(B + 1, np.int32), row_ptr=np.empty(P + 1, np.int32),
               id_map=np.empty(max(P, 1), np.int32), col=np.empty(max(g.m, 1), np.int32),
               w=np.empty(max(g.m, 1), np.int32), range_ptr=np.empty((R + 1) * B, np.int32))
    gc.tocab_export(part, out["blk_rowoff"], out["row_ptr"], out["id_map"], out["col"],
                    out["w"] if g.weights is not None else None, out["range_ptr"])
    gc.gc_sync()
    return out, B, P, R


@pytest.mark.parametrize("name", ["rmat16", "rmat17_noperm", "grid300x301", "uniform", "dangling_mix"])
@pytest.mark.parametrize("W,k", [(1 << 10, 256), (1 << 12, 4096), (1 << 14, 1024), (1 << 20, 16384)])
@pytest.mark.parametrize("direction", ["pull", "push"])
def test_partition_bit_exact(name, W, k, direction):
    import paper_1904_02241_amd as gc
    g = GRAPHS[name]().with_weights(9)
    print(f"partition {name} W={W} k={k} {direction}", flush=True)
    h = load(g, weights=True)
    d = gc.GC_PULL if direction == "pull" else gc.GC_PUSH
    part = gc.tocab_partition(h, d, W, k)
    got, B, P, R = export_partition(part, g)
    part.free()
    h.free()
    if direction == "pull":
        ar, ac, aw = oracle.transpose(g.n, g.rowptr, g.colidx, g.weights)
    else:
        ar, ac, aw = g.rowptr, g.colidx, g.weights
    want = oracle.partition(g.n, g.n, ar, ac, W, k, aw)
    assert (B, P) == (want.B, want.P)
    np.testing.assert_array_equal(got["blk_rowoff"], want.blk_rowoff)
    np.testing.assert_array_equal(got["row_ptr"], want.row_ptr)
    np.testing.assert_array_equal(got["id_map"][:P], want.id_map)
    np.testing.assert_array_equal(got["col"][:g.m], want.col)
    np.testing.assert_array_equal(got["w"][:g.m], want.w)
    np.testing.assert_array_equal(got["range_ptr"].reshape(R + 1, B).T, want.range_ptr)


def _arcs(n, m, seed):
    """A graph of exactly m arcs (distinct, no loops) over n vertices."""
    rng = np.random.default_rng(seed)
    keys = rng.choice(n * (n - 1), m, replace=False)
    u, v = keys // (n - 1), keys % (n - 1)
    return gg.from_edges(n, u, v + (v >= u), name=f"arcs{n}_{m}")


# the edges of the radix passes: one arc, a head word (64 arcs) and two arc tiles (8192) less, full and more; one
# vertex bit, digits of equal and unequal width; one block, the largest one-pass block count and two passes;
# rows and blocks far apart (long runs of empty rows)
@pytest.mark.parametrize("n,m,W,k", [(2, 1, 1 << 10, 256), (2, 2, 1 << 10, 256), (300, 63, 1 << 10, 256),
                                     (300, 64, 1 << 10, 256), (300, 65, 1 << 10, 512), (1025, 8191, 1 << 10, 256),
                                     (1025, 8192, 1 << 10, 256), (1024, 8193, 1 << 10, 256),
                                     (1 << 20, 20000, 1 << 10, 16384), ((1 << 20) + 1, 20000, 1 << 10, 16384),
                                     (3000001, 5, 1 << 11, 16384), (200000, 16385, 1 << 17, 1024)])
@pytest.mark.parametrize("direction", ["pull", "push"])
def test_radix_edges_bit_exact(n, m, W, k, direction):
    import paper_1904_02241_amd as gc
    g = _arcs(n, m, seed=m)
    g.with_weights(5)
    print(f"radix n={n} m={m} W={W} k={k} {direction}", flush=True)
    h = load(g, weights=True)
    ar, ac, aw = oracle.transpose(g.n, g.rowptr, g.colidx, g.weights)
    tr, tc, tw = np.empty(n + 1, np.int32), np.empty(m, np.int32), np.empty(m, np.int32)
    gc.graph_export_transpose(h, tr, tc, tw)
    gc.gc_sync()
    for got, want in ((tr, ar), (tc, ac), (tw, aw)):
        np.testing.assert_array_equal(got, want)
    part = gc.tocab_partition(h, gc.GC_PULL if direction == "pull" else gc.GC_PUSH, W, k)
    got, B, P, R = export_partition(part, g)
    part.free()
    h.free()
    if direction == "push":
        ar, ac, aw = g.rowptr, g.colidx, g.weights
    want = oracle.partition(n, n, ar, ac, W, k, aw)
    assert (B, P) == (want.B, want.P)
    for name in ("blk_rowoff", "row_ptr"):
        np.testing.assert_array_equal(got[name], getattr(want, name))
    np.testing.assert_array_equal(got["id_map"][:P], want.id_map)
    np.testing.assert_array_equal(got["col"], want.col)
    np.testing.assert_array_equal(got["w"], want.w)
    np.testing.assert_array_equal(got["range_ptr"].reshape(R + 1, B).T, want.range_ptr)


def test_partition_rejects_bad_widths():
    import paper_1904_02241_amd as gc
    g = gg.rmat(12, 8, seed=1)
    h = load(g)
    for W, k in [(1000, 256), (1 << 9, 256), (1 << 12, 100), (1 << 12, 1 << 15)]:
        with pytest.raises(gc.GraphCageError) as e:
            gc.tocab_partition(h, gc.GC_PULL, W, k)
        assert e.value.code == gc.GC_EINVAL
    h.free()


class _Capped:
    """The library's allocator with a limit on the bytes held (no handle may be alive outside)."""

    def __init__(self, gc):
        import torch
        self.gc, self.cap, self.live, self.peak, self.size = gc, None, 0, 0, {}

        @gc._ALLOC_FN
        def alloc(nbytes, stream, ctx):
            if self.cap is not None and self.live + nbytes > self.cap:
                return None
            p = torch.cuda.caching_allocator_alloc(int(nbytes), stream=int(stream or 0))
            self.size[p] = int(nbytes)
            self.live += int(nbytes)
            self.peak = max(self.peak, self.live)
            return p

        @gc._FREE_FN
        def release(ptr, stream, ctx):
            self.live -= self.size.pop(int(ptr))
            torch.cuda.caching_allocator_delete(int(ptr))

        self.fns = alloc, release

    def __enter__(self):
        self.gc._check(self.gc.lib.gc_set_allocator(*self.fns, None), "gc_set_allocator")
        return self

    def __exit__(self, *a):
        self.gc.use_torch_allocator(True)


def test_push_partition_leaves_the_second_layout_out_where_memory_is_short():
    """Whatever the limit: the partition as asked for where that fits, the second layout (blocks of 2^12 here)
    beside it where both do, and an error with nothing kept where the first does not."""
    import paper_1904_02241_amd as gc
    from tests.gpu_util import dev, host
    import torch
    g = gg.uniform(600007, 3000000, seed=3)
    n, W, k = g.n, 1 << 14, 4096
    with _Capped(gc) as a:
        h = gc.graph_load_csr(g.rowptr, g.colidx)
        base = a.live
        a.peak = 0
        part = gc.tocab_partition(h, gc.GC_PUSH, W, k)
        full, kept = a.peak, a.live - base
        part.free()
        assert a.live == base
        rin = dev(np.full(n, 1.0 / n, np.float32))
        want = oracle.pagerank(n, g.rowptr, g.colidx, 0.85, 3, r0=host(rin).astype(np.float64))
        sizes = []
        for cap in [full] + [base + (full - base) * i // 16 for i in range(15, 3, -1)] + [full - 1]:
            a.cap = cap
            print(f"push partition under {cap - base} of {full - base} bytes", flush=True)
            try:
                part = gc.tocab_partition(h, gc.GC_PUSH, W, k)
            except gc.GraphCageError as e:
                assert e.code == gc.GC_ENOMEM and a.live == base
                sizes.append(0)
                continue
            sizes.append(a.live - base)
            assert (part.info["W"], part.info["k"]) == (W, k)
            out = torch.empty_like(rin)
            gc.pagerank_iter(h, part, gc.GC_PULL, 0.85, 0, rin, out, 3)
            assert float(np.abs(host(out).astype(np.float64) - want).sum()) <= 1e-6
            part.free()
            assert a.live == base
        a.cap = None
        h.free()
    print(f"held {sizes}, {kept} without a limit", flush=True)
    assert sizes[0] == kept          # room for both
    assert 0 < sizes[-1] < kept      # a byte less than both take while they are built: the one asked for
    assert sizes[-2] == 0            # and too little for either


def _rows(*parts):
    return np.concatenate([np.asarray(p, np.int64) for p in parts])


# rows whose arcs are few or stand far apart: a tile of 4096 arcs over 32,768 rows (as many as it takes itself) and
# over one more, the same for the 98,304 rows that it marks, two such tiles in one run of 4096 rows, a hub before a
# gap, rows at the edges of the runs, nothing but a tail
_HOLLOW = {
    "at_limit": (40000, lambda: _rows(np.linspace(0, 32767, 4096), [39999])),
    "beyond": (40000, lambda: _rows(np.linspace(0, 32768, 4096), [39999])),
    "marks_at_limit": (110000, lambda: _rows(np.linspace(0, 98304, 4096), [109999])),
    "marks_beyond": (110000, lambda: _rows(np.linspace(0, 98305, 4096), [109999])),
    "two_tiles": (160001, lambda: _rows(np.arange(4096) * 17, 4096 * 17 + np.arange(4096) * 19, 150000 + np.arange(300))),
    "hub_gap": (300007, lambda: _rows(np.full(5000, 7), [8, 4095, 4096, 8191, 250000], np.full(4097, 299999))),
    "dense_between": (400003, lambda: _rows(np.arange(0, 100000, 50), 100000 + np.arange(9000), [399999])),
    "tail": (1000003, lambda: 1000003 - 1 - np.arange(6000)),
    "head": (1000003, lambda: np.arange(6000)),
    "few": (3000017, lambda: [4095, 4096, 12287, 2999999]),
}


@pytest.mark.parametrize("name", list(_HOLLOW))
@pytest.mark.parametrize("side", ["dst", "src"])
def test_hollow_graphs_bit_exact(name, side):
    import paper_1904_02241_amd as gc
    n, rows = _HOLLOW[name]
    a = np.asarray(rows(), np.int64)
    b = (a + 1 + np.arange(len(a)) % 6001) % n  # distinct (row, other end), no loops
    g = gg.from_edges(n, *((b, a) if side == "dst" else (a, b)), name=f"hollow_{name}").with_weights(5)
    print(f"hollow {name} {side} n={n} m={g.m}", flush=True)
    h = load(g, weights=True)
    ar, ac, aw = oracle.transpose(n, g.rowptr, g.colidx, g.weights)
    tr, tc, tw = np.empty(n + 1, np.int32), np.empty(g.m, np.int32), np.empty(g.m, np.int32)
    gc.graph_export_transpose(h, tr, tc, tw)
    gc.gc_sync()
    for got, want in ((tr, ar), (tc, ac), (tw, aw)):
        np.testing.assert_array_equal(got, want)
    for d, csr in ((gc.GC_PULL, (ar, ac, aw)), (gc.GC_PUSH, (g.rowptr, g.colidx, g.weights))):
        part = gc.tocab_partition(h, d, 1 << 14, 4096)
        got, B, P, R = export_partition(part, g)
        part.free()
        want = oracle.partition(n, n, csr[0], csr[1], 1 << 14, 4096, csr[2])
        assert (B, P) == (want.B, want.P)
        for key in ("blk_rowoff", "row_ptr"):
            np.testing.assert_array_equal(got[key], getattr(want, key))
        np.testing.assert_array_equal(got["id_map"][:P], want.id_map)
        np.testing.assert_array_equal(got["col"], want.col)
        np.testing.assert_array_equal(got["w"], want.w)
    h.free()


@pytest.mark.parametrize("where", ["head", "tail", "ends"])
def test_empty_rows_cost_no_more_in_one_run_than_spread(where):
    """16 M vertices and 10^6 arcs: among a few of them (any long run of empty rows has one work-group in front of
    it and one behind) as fast to load and to partition as spread over all, within 8 times (0.5 ms each)."""
    import time
    import torch
    import paper_1904_02241_amd as gc
    n, m, few = 1 << 24, 1000000, 1 << 16
    rng = np.random.default_rng(1)

    def ends(kind):
        x = rng.integers(0, n if kind == "spread" else few, m)
        if kind == "tail":
            return n - 1 - x
        return np.where(rng.integers(0, 2, m) == 0, x, n - 1 - x) if kind == "ends" else x

    def seconds(kind):
        g = gg.from_edges(n, ends(kind), ends(kind), name=kind)
        rp, ci = torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()
        took = []
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            h = gc.graph_load_csr(rp, ci)
            parts = [gc.tocab_partition(h, d, 1 << 15, 4096) for d in (gc.GC_PULL, gc.GC_PUSH)]
            took.append(time.perf_counter() - t0)
            for p in parts:
                p.free()
            h.free()
        return sorted(took)[1]

    base, got = seconds("spread"), seconds(where)
    print(f"empty rows {where}: {got * 1e6:.0f} us, spread {base * 1e6:.0f}", flush=True)
    assert got <= 8 * base


@pytest.mark.parametrize("m", [4095, 4096, 4097, 8191, 8192, 8193])
@pytest.mark.parametrize("n,W", [(1025, 1 << 10), (70001, 1 << 10)])
def test_radix_tile_edges_bit_exact(n, W, m):
    """One arc tile of the radix passes (4096) less one arc, full and one more, and two."""
    test_radix_edges_bit_exact(n, m, W, 256, "pull")
    test_radix_edges_bit_exact(n, m, W, 256, "push")
