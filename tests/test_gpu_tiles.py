"""Kernels that cut a level into tiles, at the sizes where a tile can go
wrong (GPU, through the C ABI): graphs of exactly a tile of entries, one
less and one more, rows longer than a tile, runs of empty rows, many graphs
in one tile; against numpy or the oracle.  All sums here are exact (unit or
dyadic weights), so the tolerance on modularity is that of its last two
divisions and the fixed-point sum: 1e-12.
"""
import numpy as np
import pytest

import gsp_inputs as gi
import oracle
import paper_2402_11454_amd as gsp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    try:
        import torch
        count = torch.cuda.device_count()
    except Exception:
        count = 0
    if count == 0:
        pytest.skip("no GPU")
    c = gsp.Context(0)
    yield c
    c.close()


def _csr(n, u, v, weighted, seed):
    """Symmetric CSR of the pairs (u, v), u != v, with dyadic weights."""
    key = np.unique(np.concatenate([u * n + v, v * n + u]))
    row, col = key // n, key % n
    off = np.searchsorted(row, np.arange(n + 1)).astype(np.int64)
    w = None
    if weighted:
        a = np.minimum(row, col) * 7919 + np.maximum(row, col) * 104729 + seed
        w = (1.0 + (a % 31) / 8.0).astype(np.float32)
    return gi.Graph(n=n, offsets=off, cols=col.astype(np.int32), weights=w)


def _path(entries, n, weighted, seed=1):
    """A path with `entries` directed entries (even), its vertices spread
    over n ids so that runs of empty rows lie between them."""
    k = entries // 2 + 1
    at = np.sort(np.random.default_rng(seed).choice(n, k, replace=False)).astype(np.int64)
    return _csr(n, at[:-1], at[1:], weighted, seed)


def _star(leaves, n, weighted, hub=3):
    v = np.setdiff1d(np.arange(leaves + 1, dtype=np.int64) + (n - leaves - 1), [hub])
    return _csr(n, np.full(v.shape, hub, np.int64), v, weighted, 5)


def _modularity(g, memb):
    w = g.weights_f64()
    row = np.repeat(np.arange(g.n), np.diff(g.offsets))
    m2 = w.sum()
    if m2 == 0:
        return 0.0
    tot = np.bincount(memb[row], weights=w, minlength=g.n)
    return float(w[memb[row] == memb[g.cols]].sum() / m2 - ((tot / m2) ** 2).sum())


TILE = 4096
CASES = {
    "tile-2": lambda w: _path(TILE - 2, 60000, w),
    "tile": lambda w: _path(TILE, 60000, w),
    "tile+2": lambda w: _path(TILE + 2, 60000, w),
    "two": lambda w: _path(2, 70000, w),
    "dense-path": lambda w: _path(3 * TILE, 3 * TILE // 2 + 1, w),
    "star": lambda w: _star(3 * TILE + 7, 90000, w),
    "rmat13": lambda w: gi.rmat_small(13, 5, weights=(1.0, 4.0) if w else None),
}


@pytest.mark.parametrize("order", [gsp.ORDER_LOADED, gsp.ORDER_DEGREE])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_modularity_at_the_tiles_edges(ctx, name, weighted, order):
    g = CASES[name](weighted)
    ctx.load_graph(g)
    if order == gsp.ORDER_DEGREE:
        ctx.run(1e-2, 1, vertex_order=order)   # builds the copy the evaluation then reads
    for ncomm in (1, 2, 37, g.n):
        m = gi.random_membership(g.n, ncomm, 11 + ncomm)
        assert abs(ctx.modularity(m) - _modularity(g, m)) <= 1e-12
        assert ctx.count_disconnected(m) == oracle.disconnected(g, m)[0]


WALK = 8 * TILE   # rows between a tile's first and last entry that are walked


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("rows", [WALK - 1, WALK, WALK + 1, 3000000])
def test_inside_weight_across_empty_rows(ctx, rows, weighted):
    """A path whose ids leave empty rows in the middle of its second tile, so
    that the tile spans `rows` rows, and of its last, which is not full; of a
    single graph and, beside others, of a batch."""
    a, b = TILE // 2, TILE   # the path's vertices that hold the second tile's first and last entry
    ids = np.arange(2 * TILE - 300, dtype=np.int64)
    ids[a + 700:] += rows - (b - a)
    ids[-500:] += rows
    n = int(ids[-1]) + 40
    g = _csr(n, ids[:-1], ids[1:], weighted, 3)
    row_of = np.repeat(np.arange(n), np.diff(g.offsets))
    assert row_of[2 * TILE - 1] - row_of[TILE] == rows
    ctx.load_graph(g)
    for m in (np.zeros(n, np.int32), (np.arange(n) // 3).astype(np.int32), gi.random_membership(n, 7, 5)):
        assert abs(ctx.modularity(m) - _modularity(g, m)) <= 1e-12
    gs = [g, _path(40, 300, weighted), g]
    ctx.load_batch(gs)
    ctx.run_batch(1e-2, 10)
    q = ctx.batch_modularity()
    for k, h in enumerate(gs):
        assert abs(q[k] - _modularity(h, ctx.batch_membership(k))) <= 1e-12


@pytest.mark.parametrize("weighted", [False, True])
def test_batch_modularity_with_many_graphs_in_a_tile(ctx, weighted):
    """Graphs of 2 to 4,098 entries side by side: several per tile, a tile
    that ends with a graph, a graph that spans tiles, graphs without entries."""
    gs = []
    for k, entries in enumerate([2, 40, 0, 4054, 4096, 0, 0, 6, 4098, 100, 8200, 2]):
        gs.append(_path(entries, 4200 + 13 * k, weighted, seed=k) if entries else
                  gi.Graph(n=5, offsets=np.zeros(6, np.int64), cols=np.zeros(0, np.int32),
                           weights=np.zeros(0, np.float32) if weighted else None))
    ctx.load_batch(gs)
    ctx.run_batch(1e-2, 10)
    q = ctx.batch_modularity()
    for k, g in enumerate(gs):
        assert abs(q[k] - _modularity(g, ctx.batch_membership(k))) <= 1e-12


@pytest.mark.parametrize("graphs", [1, 495, 496, 1500])
def test_batches_around_the_results_capacity(ctx, graphs):
    """A sweep's totals and every graph's own come back through one buffer of
    1,024 words that larger batches replace: batches on both sides of it (33
    totals, one count, two words a graph), in turn on one context, and a
    single graph after each."""
    import torch
    r = np.random.default_rng(graphs)
    gs = []
    for _ in range(graphs):
        n = int(r.integers(2, 12))
        u, v = r.integers(0, n, 2 * n), r.integers(0, n, 2 * n)
        gs.append(_csr(n, u[u != v], v[u != v], False, 0))
    ctx.load_batch(gs)
    ctx.run_batch(1e-2, 10)
    passes = ctx.batch_passes()
    for k, g in enumerate(gs):
        ref = oracle.louvain(g, 1e-2, 10, sync=True, rounds=8)
        assert np.array_equal(ctx.batch_membership(k), ref.membership), k
        assert passes[k] == ref.passes, k
    for k in {0, graphs - 1}:
        d = torch.full((gs[k].n,), -1, dtype=torch.int32, device="cuda")
        ctx._check(gsp.lib().gsp_get_batch_membership(ctx._h, k, d.data_ptr(), gsp.DEVICE), "membership")
        assert np.array_equal(d.cpu().numpy(), ctx.batch_membership(k))
    ctx.load_graph(gs[0])
    assert np.array_equal(ctx.louvain(1e-2, 10).membership,
                          oracle.louvain(gs[0], 1e-2, 10, sync=True, rounds=8).membership)


def _same_run(ctx, g, **kw):
    """A whole run equal to the oracle's: membership, passes, iterations,
    communities."""
    opt = dict(kw)
    rounds, returns = opt.get("sub_rounds", 8), bool(opt.get("return_moves", 0))
    ref = oracle.louvain(g, 1e-2, 10, sync=True, rounds=rounds, return_moves=returns)
    res = ctx.louvain(1e-2, 10, **opt)
    assert np.array_equal(res.membership, ref.membership)
    assert res.stats["passes"] == ref.passes
    assert res.stats["iterations"] == list(ref.iterations)
    assert res.stats["communities"] == list(ref.communities)
    assert res.stats["vertices"] == list(ref.vertices)
    # the counters, and the launch-by-launch run they are compared with
    slow = ctx.louvain(1e-2, 10, timing=2, **opt)
    assert np.array_equal(slow.membership, ref.membership)
    for key in ("moves", "scanned_entries", "scanned_vertices", "sweeps"):
        assert res.stats[key] == slow.stats[key]
    for kernel in ("move_small", "move_wave", "move_block"):
        assert res.stats["kernels"][kernel]["items"] == slow.stats["kernels"][kernel]["items"]
    assert abs(res.modularity - ref.modularity) <= 1e-9


@pytest.mark.parametrize("use_graphs", [0, 1])
@pytest.mark.parametrize("sub_rounds", [1, 2, 8, 64])
@pytest.mark.parametrize("n", [2, 3, 9, 300, 5000])
def test_sub_rounds_without_hubs(ctx, n, sub_rounds, use_graphs):
    """Levels without hubs apply one sub-round and compact the next in one
    launch: sub-rounds with no vertex between others, one sub-round only,
    more sub-rounds than vertices (the return-move option keeps the level's
    launches whatever its size)."""
    r = np.random.default_rng(n)
    m = 4 * n
    u, v = r.integers(0, n, m), r.integers(0, n, m)
    g = _csr(n, u[u != v], v[u != v], True, n)
    ctx.load_graph(g)
    for rm in (0, 1):
        _same_run(ctx, g, sub_rounds=sub_rounds, use_graphs=use_graphs, return_moves=rm)


@pytest.mark.parametrize("n", [163840, 163841, 300000])
@pytest.mark.parametrize("hub", [False, True])
def test_long_queues_are_applied_in_wide_tiles(ctx, n, hub):
    """One sub-round holds every vertex: queues of 163,840 entries and one
    more, where the tiles of the moves grow, and more; first every vertex in
    a community of its own (more communities than the tile's table takes),
    then communities that many movers join; with a hub and without."""
    r = np.random.default_rng(n + hub)
    u, v = r.integers(0, n, 2 * n), r.integers(0, n, 2 * n) // 40
    u, v = np.concatenate([u, np.arange(n)]), np.concatenate([v, (np.arange(n) + 1) % n])
    if hub:
        u, v = np.concatenate([u, np.zeros(6000, np.int64)]), np.concatenate([v, np.arange(1, 6001) * 17])
    g = _csr(n, u[u != v], v[u != v], hub, n)
    ctx.load_graph(g)
    ref = oracle.louvain(g, 1e-2, 3, sync=True, rounds=1)
    for kw in (dict(), dict(vertex_order=gsp.ORDER_DEGREE)):
        res = ctx.louvain(1e-2, 3, sub_rounds=1, **kw)
        assert np.array_equal(res.membership, ref.membership)
        assert res.stats["iterations"] == list(ref.iterations)


def _dense(n, p, weighted, seed, loops=False):
    """A random graph with mean degree p n; weights dyadic."""
    r = np.random.default_rng(seed)
    m = int(p * n * n / 2)
    u, v = r.integers(0, n, m), r.integers(0, n, m)
    g = _csr(n, u[u != v], v[u != v], weighted, seed)
    return gi.with_self_loops(g, {0: 2.0, n - 1: 1.5, n // 2: 0.25}) if loops else g


SMALL = {
    # the last size that one workgroup takes, and the first that it leaves
    "n1536": lambda: _dense(1536, 8 / 1536, True, 1),
    "n1537": lambda: _dense(1537, 8 / 1537, True, 2),
    "entries": lambda: _dense(1500, 42 / 1500, False, 3),
    "over": lambda: _dense(1500, 46 / 1500, False, 4),
    # up to 512 vertices every wavefront has a dense table (and four times
    # the entries fit); beyond, rows of more than 341 entries share a few
    "complete512": lambda: _dense(512, 12.0, True, 11),
    "complete513": lambda: _dense(513, 12.0, True, 12),
    "long-rows": lambda: gi.sbm(150, 1, 0.9, 0.9, 3, weights=(1.0, 4.0)),
    "hubs600": lambda: _csr(600, np.repeat(np.arange(40), 599), np.concatenate(
        [np.setdiff1d(np.arange(600), [i]) for i in range(40)]), True, 13),
    # rows around the classes' ends: 64 / 65, 341 / 342 entries, a star
    "rows64": lambda: _dense(900, 64 / 900, True, 5, loops=True),
    "rows341": lambda: gi.sbm(180, 2, 0.97, 0.9, 3, weights=(1.0, 4.0)),
    "clique": lambda: _dense(255, 3.0, True, 7),
    "star": lambda: _star(1500, 1530, True),
    "cliques": lambda: _csr(1400, *[np.array(x) for x in zip(*[(7 * c + i, 7 * c + j) for c in range(200)
                                                               for i in range(7) for j in range(i)])], True, 8),
    "path": lambda: _path(2000, 1300, True),
    "sbm1k": lambda: gi.sbm(1013, 10, 0.09, 0.004, 4),
    "sbm10k": lambda: gi.planted_sbm_10k(3),
    "road": lambda: gi.road_small(40, 3),
    "edgeless": lambda: gi.Graph(n=7, offsets=np.zeros(8, np.int64), cols=np.zeros(0, np.int32)),
    "loop": lambda: gi.Graph(n=1, offsets=np.array([0, 1]), cols=np.zeros(1, np.int32),
                             weights=np.array([2.0], np.float32)),
    "zero-weights": lambda: gi.Graph(n=4, offsets=np.array([0, 2, 4, 6, 8]),
                                     cols=np.array([1, 2, 0, 3, 0, 3, 1, 2], np.int32),
                                     weights=np.array([0, 1, 0, 0, 1, 0, 0, 0], np.float32)),
}


@pytest.mark.parametrize("sub_rounds", [1, 8, 64])
@pytest.mark.parametrize("name", list(SMALL))
def test_small_levels_in_one_launch(ctx, name, sub_rounds):
    """Levels that one workgroup takes through the rest of the run: the same
    run as the oracle's and, with the same counters, as the level-wide
    kernels'."""
    g = SMALL[name]()
    ctx.load_graph(g)
    _same_run(ctx, g, sub_rounds=sub_rounds)


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("n, sub_rounds, entries", [(700, 1, 16384), (700, 2, 32768), (700, 8, 65536),
                                                    (512, 1, 16384), (512, 8, 131072), (511, 16, 260610)])
def test_small_levels_at_the_entries_limit(ctx, n, sub_rounds, entries, over):
    """Exactly as many entries as one workgroup takes in a run with so many
    sub-rounds, and two more (the last pair: a complete graph, and one edge
    short of it)."""
    u, v = np.triu_indices(n, 1)
    m = min(entries // 2 + over, u.shape[0] - (1 - over))
    k = np.random.default_rng(n + entries).permutation(u.shape[0])[:m]
    g = _csr(n, u[k].astype(np.int64), v[k].astype(np.int64), True, entries)
    ctx.load_graph(g)
    _same_run(ctx, g, sub_rounds=sub_rounds)


@pytest.mark.parametrize("kw", [dict(max_iterations=0), dict(max_iterations=1), dict(aggregation_tolerance=0.3),
                                dict(aggregation_tolerance=1.0), dict(tolerance_drop=2.0)])
@pytest.mark.parametrize("max_passes", [1, 2, 10])
def test_small_levels_options(ctx, kw, max_passes):
    g = SMALL["sbm1k"]()
    ctx.load_graph(g)
    ref = oracle.louvain(g, 1e-2, max_passes, sync=True, rounds=8, **kw)
    res = ctx.louvain(1e-2, max_passes, **kw)
    assert np.array_equal(res.membership, ref.membership)
    assert res.stats["iterations"] == list(ref.iterations)
    assert res.stats["communities"] == list(ref.communities)


def test_small_graph_with_duplicates_and_fp64_weights(ctx):
    """Rows that hold a column twice, fp64 weights that need the grid."""
    r = np.random.default_rng(9)
    n, m = 400, 3000
    u, v = r.integers(0, n, m), r.integers(0, n, m)
    w = r.uniform(0.1, 3.0, m)
    row, col, ww = np.concatenate([u, v]), np.concatenate([v, u]), np.concatenate([w, w])
    keep = row != col
    order = np.argsort(row[keep], kind="stable")
    row, col, ww = row[keep][order], col[keep][order].astype(np.int32), ww[keep][order]
    off = np.searchsorted(row, np.arange(n + 1)).astype(np.int64)
    ctx.load(off, col, ww)
    wg = ww.copy()
    assert oracle.weight_grid(wg)[0] == ctx.weight_grid()[0]
    g = oracle.CSR(n, off, col, wg)
    ref = oracle.louvain(g, 1e-2, 10, sync=True, rounds=8)
    assert np.array_equal(ctx.louvain(1e-2, 10).membership, ref.membership)


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 5000])
def test_aggregation_counts_at_the_tiles_edges(ctx, n):
    """Members and degrees are counted in one word per community by tiles of
    1,024 vertices: one vertex, a tile less one and more, several tiles;
    communities of isolated vertices only, of both kinds, one for all."""
    r = np.random.default_rng(n)
    ends = r.choice(n, max(2, n // 2)) if n > 1 else np.zeros(2, np.int64)
    u, v = r.choice(ends, 3 * n), r.choice(ends, 3 * n)   # half of the vertices have no entries
    g = _csr(n, u[u != v].astype(np.int64), v[u != v].astype(np.int64), True, n)
    ctx.load_graph(g)
    for m in (np.zeros(n, np.int32), np.arange(n, dtype=np.int32), r.integers(0, max(1, n // 7), n).astype(np.int32),
              np.where(np.diff(g.offsets) > 0, 0, n - 1).astype(np.int32)):
        mr, G = oracle.renumber(m)
        ref = oracle.aggregate(g, mr, G)
        n2, off, col, w = ctx.step_aggregate(m)
        assert n2 == G
        assert np.array_equal(off, ref.off)
        for c in range(n2):
            a, b = slice(int(off[c]), int(off[c + 1])), slice(int(ref.off[c]), int(ref.off[c + 1]))
            o, q = np.argsort(col[a]), np.argsort(ref.col[b])
            assert np.array_equal(col[a][o], ref.col[b][q]) and np.array_equal(w[a][o], ref.w[b][q])


@pytest.mark.parametrize("n", [2, 7, 8, 63, 64, 65, 513, 4097])
def test_degree_order_label_minima(ctx, n):
    """The smallest caller's id of each community in degree order, taken over
    a 64th, an eighth and the rest of the vertices: sizes where these are
    empty or one vertex (a whole run, one pass and several)."""
    r = np.random.default_rng(n)
    u, v = r.integers(0, n, 5 * n), r.integers(0, n, 5 * n)
    g = _csr(n, u[u != v], v[u != v], True, n)
    ctx.load_graph(g)
    for passes in (1, 10):
        ref = oracle.louvain(g, 1e-2, passes, sync=True, rounds=8)
        assert np.array_equal(ctx.louvain(1e-2, passes, vertex_order=gsp.ORDER_DEGREE).membership, ref.membership)


@pytest.mark.parametrize("n", [524287, 524288, 526337])
@pytest.mark.parametrize("communities", [1, 4000, 4097, 300000])
def test_community_totals_in_kept_tables(ctx, n, communities):
    """From 524,288 vertices on a workgroup keeps its table of 8,192 slots over
    several tiles and empties it when half of them are taken: one community,
    as many as never fill half, just more, and more in a tile than half."""
    r = np.random.default_rng(n + communities)
    g = _csr(n, np.arange(n - 1, dtype=np.int64), np.arange(1, n, dtype=np.int64), True, n)
    m = r.integers(0, communities, n).astype(np.int32)
    ctx.load_graph(g)
    assert abs(ctx.modularity(m) - _modularity(g, m)) <= 1e-12


@pytest.mark.parametrize("communities", [1, 6000, 200000, 2700001])
def test_community_totals_emptied_in_mid_range(ctx, communities):
    """Five or six tiles of 2,048 vertices per workgroup: any three of them
    hold more communities than half a table, so it is emptied and used again
    before the last (6,000: once or twice; more: every third tile).  Totals by
    the modularity, totals and sizes by a step's decisions (a third of the
    vertices alone in their communities)."""
    n = 2700001
    r = np.random.default_rng(communities)
    g = _csr(n, np.arange(n - 1, dtype=np.int64), np.arange(1, n, dtype=np.int64), True, n)
    ctx.load_graph(g)
    m = r.integers(0, communities, n).astype(np.int32)
    assert abs(ctx.modularity(m) - _modularity(g, m)) <= 1e-12
    if communities < n:
        alone = np.flatnonzero(r.integers(0, 3, n) == 0)
        m[alone[alone >= communities]] = alone[alone >= communities]
    dec, gain, moved = ctx.step_move(m)
    ref = oracle.move_sync_step(g, m)
    assert np.array_equal(dec, ref[0])


@pytest.mark.parametrize("n, sub_rounds", [(524288, 8), (524289, 8), (524289, 64), (530001, 1)])
def test_work_lists_in_wide_tiles(ctx, n, sub_rounds):
    """Above 524,288 vertices the work lists are filled in tiles of 4,096."""
    r = np.random.default_rng(n)
    u, v = r.integers(0, n, n), r.integers(0, n, n) // 9
    g = _csr(n, u[u != v], v[u != v], False, 0)
    ctx.load_graph(g)
    ref = oracle.louvain(g, 1e-2, 1, sync=True, rounds=sub_rounds)
    res = ctx.louvain(1e-2, 1, sub_rounds=sub_rounds, vertex_order=gsp.ORDER_LOADED)
    assert np.array_equal(res.membership, ref.membership)


@pytest.mark.parametrize("n", [524287, 524288, 600001])
@pytest.mark.parametrize("communities", [1, 4097, 60000, 300000])
def test_aggregation_counts_in_kept_tables(ctx, n, communities):
    """From 524,288 vertices on a workgroup keeps its table of communities over
    the tiles of its range and places the vertices when it empties it: row
    totals of the aggregated graph against numpy (exact weights)."""
    r = np.random.default_rng(n + communities)
    i = np.arange(n // 2 - 1, dtype=np.int64)   # the second half has no entries
    g = _csr(n, i, i + 1, True, n)
    m = r.integers(0, communities, n).astype(np.int32)
    ctx.load_graph(g)
    n2, off, col, w = ctx.step_aggregate(m)
    used, mr = np.unique(m, return_inverse=True)
    assert n2 == used.shape[0]
    row = np.repeat(np.arange(n), np.diff(g.offsets))
    key, at = np.unique(mr[row].astype(np.int64) * n2 + mr[g.cols], return_inverse=True)
    ref = np.bincount(at, weights=g.weights_f64())
    got = np.repeat(np.arange(n2), np.diff(off)) * np.int64(n2) + col
    o = np.argsort(got)
    assert np.array_equal(got[o], key) and np.array_equal(w[o], ref)


@pytest.mark.parametrize("communities", [6000, 200000, 330000])
def test_aggregation_counts_emptied_in_mid_range(ctx, communities):
    """Six tiles of 2,048 vertices per workgroup: its table is emptied, and the
    vertices placed, before the last tile and again after (6,000 communities:
    about every fourth tile; more: every third): members, degrees and row
    totals of the aggregated graph against numpy (exact weights)."""
    n = 2700001
    r = np.random.default_rng(communities)
    i = np.arange(n - 1, dtype=np.int64)[r.integers(0, 3, n - 1) > 0]   # some vertices have no entries
    g = _csr(n, i, i + 1, True, n)
    m = r.integers(0, communities, n).astype(np.int32)
    ctx.load_graph(g)
    n2, off, col, w = ctx.step_aggregate(m)
    used, mr = np.unique(m, return_inverse=True)
    assert n2 == used.shape[0]
    row = np.repeat(np.arange(n), np.diff(g.offsets))
    key, at = np.unique(mr[row].astype(np.int64) * n2 + mr[g.cols], return_inverse=True)
    ref = np.bincount(at, weights=g.weights_f64())
    got = np.repeat(np.arange(n2), np.diff(off)) * np.int64(n2) + col
    o = np.argsort(got)
    assert np.array_equal(got[o], key) and np.array_equal(w[o], ref)


def test_contexts_in_threads(ctx):
    """Each context waits on a buffer of its own: four threads with a context
    and a stream each, running side by side, repeat the oracle's results."""
    import threading
    gs = [gi.rmat_small(12, 5), gi.planted_sbm_10k(), _dense(300, 0.2, True, 3), _path(20000, 12000, False)]
    want = [oracle.louvain(g, 1e-2, 10, sync=True, rounds=8).membership for g in gs]
    bad = []

    def work(k):
        try:
            c = gsp.Context(0)
            for _ in range(5):
                for q in (k, (k + 1) % len(gs)):
                    c.load_graph(gs[q])
                    if not np.array_equal(c.louvain(1e-2, 10).membership, want[q]):
                        bad.append((k, q))
            c.load_batch(gs)
            c.run_batch(1e-2, 10)
            bad.extend((k, "batch", q) for q in range(len(gs))
                       if not np.array_equal(c.batch_membership(q), want[q]))
            c.close()
        except Exception as e:   # reported below, in the test's own thread
            bad.append((k, repr(e)))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(100)
    assert not any(t.is_alive() for t in threads) and not bad
