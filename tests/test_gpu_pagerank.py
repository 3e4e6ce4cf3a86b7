"""GPU PageRank parity against the FP64 oracle: L1 <= 1e-6 after 20
iterations (plain pull, plain push, TOCAB pull, TOCAB push)."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from tests import graphs
from tests.gpu_util import load, pagerank_gpu

pytestmark = pytest.mark.gpu

L1_TOL = 1e-6
FORMS = ["plain_pull", "plain_push", "tocab_pull", "tocab_push"]


def l1(a, b):
    return float(np.abs(a.astype(np.float64) - b).sum())


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("mode", [oracle.UNIFORM, oracle.LEAK])
def test_pagerank_rmat16_20_iterations(form, mode):
    g = gg.rmat(16, 16, seed=1)
    print(f"pagerank rmat16 {form} mode={mode}", flush=True)
    got, r0 = pagerank_gpu(g, form, mode)
    want = oracle.pagerank(g.n, g.rowptr, g.colidx, 0.85, 20, mode=mode, r0=r0)
    err = l1(got, want)
    print(f"L1 = {err:.3e}")
    assert err <= L1_TOL
    if mode == oracle.UNIFORM:
        assert abs(got.astype(np.float64).sum() - 1.0) < 1e-5


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("W,k", [(1 << 10, 256), (1 << 12, 4096), (1 << 14, 16384), (1 << 15, 2048),
                                 (1 << 15, 16384), (1 << 13, 256), (1 << 17, 512)])
def test_pagerank_ragged_grid_block_shapes(form, W, k):
    g = gg.grid(300, 301, 0.05, seed=3)  # n = 90300: ragged last block and range
    print(f"pagerank grid {form} W={W} k={k}", flush=True)
    got, r0 = pagerank_gpu(g, form, oracle.UNIFORM, W=W, k=k)
    want = oracle.pagerank(g.n, g.rowptr, g.colidx, 0.85, 20, r0=r0)
    assert l1(got, want) <= L1_TOL


@pytest.mark.parametrize("g", graphs.all_small(), ids=lambda g: g.name)
@pytest.mark.parametrize("form", FORMS)
def test_pagerank_small_graphs(g, form):
    got, r0 = pagerank_gpu(g, form, oracle.UNIFORM, iters=7)
    want = oracle.pagerank(g.n, g.rowptr, g.colidx, 0.85, 7, r0=r0)
    assert l1(got, want) <= L1_TOL


@pytest.mark.parametrize("form", FORMS)
def test_pagerank_hub_rows_longer_than_a_tile(form):
    """In-rows of 8999 and 20000 arcs: the whole-work-group path of a pull
    tile, inside one block (W = 2^14 >= n) and split over blocks (W = 2^10)."""
    for g in (graphs.star_in(9000), graphs.star_in(20001)):
        for W in (1 << 14, 1 << 10, 1 << 16):
            got, r0 = pagerank_gpu(g, form, oracle.UNIFORM, iters=5, W=W, k=1024)
            want = oracle.pagerank(g.n, g.rowptr, g.colidx, 0.85, 5, r0=r0)
            assert l1(got, want) <= L1_TOL


@pytest.mark.parametrize("form", FORMS)
def test_pagerank_zero_and_one_iteration_and_custom_start(form):
    g = gg.rmat(12, 16, seed=5)
    rng = np.random.default_rng(3)
    r0 = rng.random(g.n).astype(np.float32)
    r0 /= r0.sum()
    got0, used = pagerank_gpu(g, form, oracle.UNIFORM, iters=0, r0=r0)
    np.testing.assert_array_equal(got0, r0.astype(np.float32))
    got1, used = pagerank_gpu(g, form, oracle.UNIFORM, iters=1, r0=r0)
    want1 = oracle.pagerank(g.n, g.rowptr, g.colidx, 0.85, 1, r0=used)
    assert l1(got1, want1) <= L1_TOL


def test_pagerank_chained_calls_continue_the_iteration():
    """20 iterations in one call equal 5 calls of 4 (the state is the rank)."""
    import paper_1904_02241_amd as gc
    from tests.gpu_util import dev, host, torch
    g = gg.rmat(14, 16, seed=2)
    h = load(g)
    part = gc.tocab_partition(h, gc.GC_PULL, 1 << 11, 1024)
    t = torch()
    a = dev(np.full(g.n, 1.0 / g.n, np.float32))
    b = t.empty_like(a)
    for _ in range(5):
        gc.pagerank_iter(h, part, gc.GC_PULL, 0.85, 0, a, b, 4)
        a, b = b, a
    got = host(a)
    want = oracle.pagerank(g.n, g.rowptr, g.colidx, 0.85, 20, r0=np.full(g.n, np.float32(1.0 / g.n), np.float64))
    assert l1(got, want) <= L1_TOL
    part.free()
    h.free()


# the one-work-group form of small graphs: one vertex, waves and row groups
# of every width less, full and more, rows taken by a group and by a wave
# (star: one row of all arcs), an even and an odd number of iterations, and
# graphs just inside and just outside the LDS it may take. FP32 rounding of
# ranks and contributions gives at most 2 * 2^-24 / (1 - 0.85) = 8e-7 in L1.
@pytest.mark.parametrize("make", [lambda: graphs.edgeless(1), lambda: graphs.cycle(63), lambda: graphs.cycle(64),
                                  lambda: graphs.cycle(65), lambda: graphs.cycle(257), lambda: graphs.star_in(2000),
                                  lambda: graphs.star_out(130), lambda: gg.uniform(1025, 1025 * 4, seed=2),
                                  lambda: gg.uniform(700, 700 * 12, seed=3), lambda: gg.rmat(11, 16, seed=4),
                                  lambda: gg.uniform(4000, 24000, seed=5), lambda: gg.uniform(4000, 25000, seed=5)],
                         ids=["one", "c63", "c64", "c65", "c257", "star_in", "star_out", "deg8", "deg24", "rmat11",
                              "inside", "outside"])
@pytest.mark.parametrize("form,iters", [("plain_pull", 1), ("plain_push", 2), ("tocab_pull", 7)])
def test_pagerank_one_work_group(make, form, iters):
    g = make()
    print(f"small pagerank {g.name} n={g.n} m={g.m} {form} iters={iters}", flush=True)
    for mode in (oracle.UNIFORM, oracle.LEAK):
        got, r0 = pagerank_gpu(g, form, mode, iters=iters)
        want = oracle.pagerank(g.n, g.rowptr, g.colidx, 0.85, iters, mode=mode, r0=r0)
        assert l1(got, want) <= L1_TOL


@pytest.mark.parametrize("make,W,k", [(lambda: graphs.star_out(70000), 1 << 13, 256),
                                      (lambda: gg.uniform(5000, 4095, seed=1), 1 << 12, 256),
                                      (lambda: gg.uniform(5000, 40960, seed=2), 1 << 13, 256),
                                      (lambda: gg.uniform(230001, 3 * 230001, seed=3), 1 << 15, 256),
                                      (lambda: gg.uniform(270000, 2 * 270000, seed=4), 1 << 10, 1024),
                                      (lambda: gg.rmat(16, 16, seed=5, permute=False), 1 << 10, 256)],
                         ids=["empty_blocks", "below_least", "one_block", "range_cap", "many_blocks", "skewed"])
def test_pagerank_chunk_cuts(make, W, k):
    """Chunk sizes: blocks without arcs, fewer arcs than the least chunk, one
    block, more ranges than a chunk's table holds (899 against 828), more
    blocks than CUs, blocks of very different sizes."""
    g = make()
    print(f"chunk cuts {g.name} n={g.n} m={g.m} W={W} k={k}", flush=True)
    got, r0 = pagerank_gpu(g, "tocab_pull", oracle.LEAK, iters=3, W=W, k=k)
    want = oracle.pagerank(g.n, g.rowptr, g.colidx, 0.85, 3, mode=oracle.LEAK, r0=r0)
    assert l1(got, want) <= L1_TOL


@pytest.mark.parametrize("n", [255, 16385, 32768, 130000, 2 * 127 * 1024 + 1, 128 * 2048])
@pytest.mark.parametrize("W,k", [(1 << 13, 256), (1 << 13, 2048), (1 << 13, 16384), (1 << 16, 512), (1 << 16, 2048),
                                 (1 << 16, 16384)])
def test_pagerank_split_merge_ranges(n, W, k):
    """Merge ranges as wide as given, halved once, or down to the least width."""
    g = gg.uniform(n, 6 * n, seed=n)
    print(f"split ranges n={n} W={W} k={k}", flush=True)
    got, r0 = pagerank_gpu(g, "tocab_pull", oracle.UNIFORM, iters=2, W=W, k=k)
    want = oracle.pagerank(g.n, g.rowptr, g.colidx, 0.85, 2, r0=r0)
    assert l1(got, want) <= L1_TOL


@pytest.mark.parametrize("n,W,k", [(9000, 1 << 14, 16384), (16385, 1 << 11, 256), (127 * 1024, 1 << 10, 1024),
                                   (128 * 1024 + 1, 1 << 14, 4096), (300001, 1 << 13, 256),
                                   (2100000, 1 << 11, 1024)])
@pytest.mark.parametrize("mode", [oracle.UNIFORM, oracle.LEAK])
def test_pagerank_push_inner_blocks(n, W, k, mode):
    """Push over narrower and wider blocks than the partition's: the least
    width, one short of enough blocks, ranges wider than the inner blocks; and
    the partition itself is still as asked for."""
    import paper_1904_02241_amd as gc
    g = gg.uniform(n, 5 * n, seed=n)
    print(f"push inner n={n} W={W} k={k} mode={mode}", flush=True)
    got, r0 = pagerank_gpu(g, "tocab_push", mode, iters=3, W=W, k=k)
    want = oracle.pagerank(g.n, g.rowptr, g.colidx, 0.85, 3, mode=mode, r0=r0)
    assert l1(got, want) <= L1_TOL
    h = load(g)
    part = gc.tocab_partition(h, gc.GC_PUSH, W, k)
    assert (part.info["W"], part.info["k"], part.info["B"]) == (W, k, (n + W - 1) // W)
    part.free()
    h.free()


def test_pagerank_rejects_overlap_and_bad_args():
    import paper_1904_02241_amd as gc
    from tests.gpu_util import torch
    t = torch()
    g = gg.rmat(10, 8, seed=1)
    h = load(g)
    buf = t.zeros(2 * g.n, dtype=t.float32, device="cuda")
    with pytest.raises(gc.GraphCageError):
        gc.pagerank_iter(h, None, gc.GC_PULL, 0.85, 0, buf[: g.n], buf[g.n // 2: g.n // 2 + g.n], 1)
    with pytest.raises(gc.GraphCageError):
        gc.pagerank_iter(h, None, gc.GC_PULL, 1.5, 0, buf[: g.n], buf[g.n:], 1)
    with pytest.raises(gc.GraphCageError):
        gc.pagerank_iter(h, None, 7, 0.85, 0, buf[: g.n], buf[g.n:], 1)
    h.free()


@pytest.mark.timeout(900)
def test_pagerank_rmat22_tocab_and_plain():
    g = gg.rmat(22, 16, seed=1)
    print(f"pagerank rmat22 n={g.n} m={g.m}", flush=True)
    want = None
    for form, W in [("tocab_pull", 1 << 18), ("plain_pull", 0), ("tocab_push", 1 << 18)]:
        got, r0 = pagerank_gpu(g, form, oracle.UNIFORM, W=max(W, 1 << 10), k=4096)
        if want is None:
            want = oracle.pagerank(g.n, g.rowptr, g.colidx, 0.85, 20, r0=r0)
        err = l1(got, want)
        print(f"{form}: L1 = {err:.3e}", flush=True)
        assert err <= L1_TOL


def test_autotune_picks_a_valid_width_and_caches_it():
    import paper_1904_02241_amd as gc
    g = gg.rmat(16, 16, seed=1)
    h = load(g)
    W, k, ms = gc.tocab_autotune(h, gc.GC_PULL)
    assert W & (W - 1) == 0 and (1 << 12) <= W <= (1 << 16)
    assert k in (2048, 4096, 8192) and ms > 0
    assert gc.tocab_autotune(h, gc.GC_PULL) == (W, k, ms)  # cached for this graph
    part = gc.tocab_partition(h, gc.GC_PULL, 0, 0)  # width 0: autotuned
    assert (part.info["W"], part.info["k"]) == (W, k)
    got, r0 = pagerank_gpu(g, "tocab_pull", oracle.UNIFORM, handles={"g": h}, W=W, k=k)
    want = oracle.pagerank(g.n, g.rowptr, g.colidx, 0.85, 20, r0=r0)
    assert l1(got, want) <= L1_TOL
    part.free()
    h.free()


def _exact(n, m, seed, isolated=0):
    """A graph of exactly m arcs (distinct, no loops) among n vertices, and `isolated` more."""
    rng = np.random.default_rng(seed)
    keys = rng.choice(n * (n - 1), m, replace=False)
    u, v = keys // (n - 1), keys % (n - 1)
    return gg.from_edges(n + isolated, u, v + (v >= u), name=f"arcs{n}_{m}")


def _ran(gc, call):
    """The kernels that call() launches."""
    gc.gc_profile(True)
    call()
    gc.gc_profile(False)
    return set(gc.gc_profile_read())


LDS = 158 * 1024  # what the one-work-group form may take: 18 n + 2 m + 1028 bytes, 22 n until converged


# the last graph that fits the LDS, bit for bit on its edge, and one arc more; 20 iterations and an odd number
@pytest.mark.parametrize("n", [3000, 5001, 700])
@pytest.mark.parametrize("conv", [False, True])
def test_pagerank_one_work_group_lds_edge(n, conv):
    import paper_1904_02241_amd as gc
    from tests.gpu_util import dev, host, torch
    per = 22 if conv else 18
    m = (LDS - 1028 - per * n) // 2
    assert per * n + 2 * m + 1028 == LDS
    for arcs, fits in ((m, True), (m + 1, False)):
        g = _exact(n, arcs, seed=n)
        print(f"lds edge n={n} m={g.m} conv={conv} fits={fits}", flush=True)
        h = load(g)
        rin = dev(np.full(n, 1.0 / n, np.float32))
        out = torch().empty_like(rin)
        for iters in (20, 21):
            if conv:
                ran = _ran(gc, lambda: gc.pagerank_converge(h, None, gc.GC_PUSH, 0.85, 0, rin, out, 0.0, iters))
            else:
                ran = _ran(gc, lambda: gc.pagerank_iter(h, None, gc.GC_PUSH, 0.85, 0, rin, out, iters))
            assert ("pr_small" in ran) == fits, ran
            want = oracle.pagerank(n, g.rowptr, g.colidx, 0.85, iters, r0=host(rin).astype(np.float64))
            assert l1(host(out), want) <= L1_TOL
        h.free()


# which calls take the one-work-group form: (n, arcs, form, iterations) well on either side of the line (both sides'
# times stand at the rule); the result is the same on both
@pytest.mark.parametrize("n,m,form,iters,small", [
    (1000, 8000, "plain_pull", 20, True), (3000, 48000, "plain_pull", 20, False), (500, 70000, "plain_pull", 20, False),
    (300, 70000, "tocab_pull", 20, False), (6000, 24000, "plain_pull", 20, False), (8500, 850, "plain_pull", 20, True),
    (8500, 850, "plain_push", 20, False), (8500, 850, "tocab_push", 20, False), (3000, 48000, "plain_push", 20, True),
    (1000, 60000, "tocab_push", 20, True), (3000, 24000, "tocab_pull", 20, True), (4000, 16000, "plain_pull", 1, False),
    (8000, 8000, "tocab_push", 1, False), (600, 4800, "plain_pull", 1, True)])
def test_pagerank_one_work_group_where_it_pays(n, m, form, iters, small):
    import paper_1904_02241_amd as gc
    from tests.gpu_util import dev, host, torch
    g = _exact(n, m, seed=n + m)
    print(f"one work-group n={n} m={m} {form} iters={iters}", flush=True)
    h = load(g)
    part = None
    if form.startswith("tocab"):
        part = gc.tocab_partition(h, gc.GC_PULL if form == "tocab_pull" else gc.GC_PUSH, 1 << 12, 1024)
    rin = dev(np.full(n, 1.0 / n, np.float32))
    out = torch().empty_like(rin)
    d = gc.GC_PUSH if form == "plain_push" else gc.GC_PULL
    ran = _ran(gc, lambda: gc.pagerank_iter(h, part, d, 0.85, 1, rin, out, iters))
    assert ("pr_small" in ran) == small, ran
    want = oracle.pagerank(n, g.rowptr, g.colidx, 0.85, iters, mode=oracle.LEAK, r0=host(rin).astype(np.float64))
    assert l1(host(out), want) <= L1_TOL
    if part is not None:
        part.free()
    h.free()


# rows summed by a thread or by a wave: tiles of rows all just under, at and over either line, of rows on both sides
# of it, of few rows and of many, and short rows among long ones
@pytest.mark.parametrize("rows", [(32,), (33,), (80,), (81,), (128, 129), (31, 300), (0, 1, 2000, 5), (64,), (4096, 4097),
                                  (1, 130, 0)], ids=lambda r: "-".join(map(str, r)))
@pytest.mark.parametrize("form", ["plain_pull", "tocab_wide"])
def test_pagerank_tile_rows_by_thread_and_wave(rows, form):
    import paper_1904_02241_amd as gc
    from tests.gpu_util import dev, host, torch
    n, live = 20011, min(1500, 300000 // max(rows))
    deg = np.array([rows[i % len(rows)] for i in range(live)])
    dst = np.repeat(np.arange(live), deg)
    src = (dst + 1 + np.arange(len(dst)) - np.repeat(np.cumsum(deg) - deg, deg)) % n
    g = gg.from_edges(n, src, dst, name="tile_rows")
    print(f"tile rows {rows} {form} m={g.m}", flush=True)
    h = load(g)
    part = gc.tocab_partition(h, gc.GC_PULL, 1 << 16, 256) if form == "tocab_wide" else None
    rin = dev(np.full(n, 1.0 / n, np.float32))
    out = torch().empty_like(rin)
    gc.pagerank_iter(h, part, gc.GC_PULL, 0.85, 0, rin, out, 3)
    want = oracle.pagerank(n, g.rowptr, g.colidx, 0.85, 3, r0=host(rin).astype(np.float64))
    assert l1(host(out), want) <= L1_TOL
    if part is not None:
        part.free()
    h.free()


def test_autotune_does_not_choose_between_widths_that_run_alike():
    """Push partitions of 2^12 to 2^14 run PageRank over blocks of one width, and a graph that runs as one work-group
    over none: the width that needs no second layout, or the least, is chosen, not the one noise favours."""
    import paper_1904_02241_amd as gc
    for seed in range(4):
        for n, m, directions, alike in ((600007 + seed, 3000000, (gc.GC_PUSH,), (1 << 12, 1 << 13, 1 << 14)),
                                        (5000 + seed, 10000, (gc.GC_PULL, gc.GC_PUSH), (1 << 12, 1 << 13))):
            h = load(gg.uniform(n, m, seed=seed))
            for d in directions:
                W, k, ms = gc.tocab_autotune(h, d)
                print(f"autotune n={n} dir={d}: {W} {k} {ms:.4f}", flush=True)
                assert W == alike[0] or W not in alike
                assert ms > 0
            h.free()


# the corner shapes of the small graphs, padded with isolated vertices past what one work-group holds, so that the
# tiled, pushed and blocked kernels meet them: no arc, one row or one column of all arcs, chains, sinks
@pytest.mark.parametrize("make", [lambda: graphs.edgeless(5), lambda: graphs.star_out(9), lambda: graphs.star_in(9),
                                  lambda: graphs.star_in(5001), lambda: graphs.star_out(9000), lambda: graphs.chain(8),
                                  lambda: graphs.chain(3000), lambda: graphs.complete(6), lambda: graphs.dangling_mix(),
                                  lambda: graphs.two_components(), lambda: graphs.random_small(40, 120, 1)],
                         ids=["edgeless", "star_out9", "star_in9", "star_in5001", "star_out9000", "chain8", "chain3000",
                              "complete", "dangling_mix", "two_components", "random"])
@pytest.mark.parametrize("form", FORMS + ["tocab_wide"])
def test_pagerank_corner_shapes_beyond_one_work_group(make, form):
    import paper_1904_02241_amd as gc
    from tests.gpu_util import dev, host, torch
    small = make()
    n = 20011
    src = np.repeat(np.arange(small.n), np.diff(small.rowptr))
    for shift in (0, n - small.n):  # the shape among the first vertices, and among the last
        g = gg.from_edges(n, src + shift, small.colidx.astype(np.int64) + shift, name=f"{small.name}_padded")
        h = load(g)
        part = None
        if form.startswith("tocab"):
            part = gc.tocab_partition(h, gc.GC_PUSH if form == "tocab_push" else gc.GC_PULL,
                                      1 << 16 if form == "tocab_wide" else 1 << 11, 256)
        rin = dev(np.full(n, 1.0 / n, np.float32))
        out = torch().empty_like(rin)
        d = gc.GC_PUSH if form == "plain_push" else gc.GC_PULL
        for mode in (oracle.UNIFORM, oracle.LEAK):
            print(f"padded {small.name} {form} shift={shift} mode={mode}", flush=True)
            ran = _ran(gc, lambda: gc.pagerank_iter(h, part, d, 0.85, mode, rin, out, 5))
            assert "pr_small" not in ran
            want = oracle.pagerank(n, g.rowptr, g.colidx, 0.85, 5, mode=mode, r0=host(rin).astype(np.float64))
            assert l1(host(out), want) <= L1_TOL
        if part is not None:
            part.free()
        h.free()
