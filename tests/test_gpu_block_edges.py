"""Batch kernels at the edges of their blocks and grids, against the oracle."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import paper_2507_11094_amd as m
    return m


# one element, around one 1,024-thread block, around the 512 resident blocks
@pytest.mark.parametrize("k", [1, 2, 1023, 1024, 1025, 2049, 524287, 524289])
def test_batch_counts_and_distances(dg, k):
    n, s, d, w = graphgen.rmat_directed(16, 1 << 20, graphgen.config_seed(0, 41))
    b = graphgen.update_batch(n, s, d, k, graphgen.config_seed(0, 42 + k))
    G = dg.Graph(n, s, d, w)
    qs = G.sssp_attach(0)
    qp = G.pr_attach(0.85, 1e-9, 1000)
    st = G.apply(*b)
    assert (st.deleted, st.inserted) == (k // 2, k - k // 2)
    s2, d2, w2, _ = oracle.apply(n, s, d, w, *b)
    assert np.array_equal(qs.read()[0], oracle.sssp(n, s2, d2, w2, 0))
    want, _, _ = oracle.pagerank(n, s2, d2, 0.85, 1e-9, 1000)
    assert np.max(np.abs(qp.read()[0] - want)) <= 1e-10
    # one self-loop anywhere rejects the whole batch
    bad = [x.copy() for x in b]
    bad[0][k - 1] = bad[1][k - 1]
    with pytest.raises(dg.DGError):
        G.apply(*bad)
    assert np.array_equal(qs.read()[0], oracle.sssp(n, s2, d2, w2, 0))
    G.close()


# frontiers and rows around a wave's slots, the heavy degree and the wave-count rule
@pytest.mark.parametrize("heavy,delta", [(0, 0), (64, 0), (0, 30)])
@pytest.mark.parametrize("k", [1, 7, 8, 9, 63, 65, 255, 257, 511, 513, 16383, 16385])
def test_frontier_shapes(dg, k, heavy, delta):
    rng = np.random.default_rng(k)
    # 0 -> k middle vertices -> three of seven sinks each, and one sink back to all
    mid = np.arange(1, k + 1)
    s = np.concatenate([np.zeros(k, np.int64), np.repeat(mid, 3), np.full(k, k + 1)])
    d = np.concatenate([mid, k + 1 + (mid[:, None] + np.arange(3)).ravel() % 7, mid])
    w = rng.integers(1, 50, s.size)
    n = k + 9
    s, d, w = s.astype(np.int32), d.astype(np.int32), w.astype(np.int32)
    c = dg.Config()
    c.heavy_degree = heavy
    c.sssp_delta = delta  # 30: near frontier and far pile
    G = dg.Graph(n, s, d, w, config=c)
    q = G.sssp_attach(0)
    assert np.array_equal(q.read()[0], oracle.sssp(n, s, d, w, 0))
    # cut half of the source's row, lengthen every third middle vertex's by a new head
    cut = rng.random(k) < 0.5
    cut[0] = True
    far = mid[::3]
    bs = np.concatenate([np.zeros(cut.sum(), np.int64), far]).astype(np.int32)
    bd = np.concatenate([mid[cut], np.full(far.size, k + 8)]).astype(np.int32)
    bo = np.concatenate([np.zeros(cut.sum()), np.ones(far.size)]).astype(np.uint8)
    bw = rng.integers(1, 50, bs.size).astype(np.int32)
    G.apply(bs, bd, bw, bo)
    s2, d2, w2, _ = oracle.apply(n, s, d, w, bs, bd, bw, bo)
    assert np.array_equal(q.read()[0], oracle.sssp(n, s2, d2, w2, 0))
    back = np.where(bo == 0, w[np.minimum(np.maximum(bd - 1, 0), k - 1)], bw).astype(np.int32)
    G.apply(bs, bd, back, 1 - bo)
    assert np.array_equal(q.read()[0], oracle.sssp(n, s, d, w, 0))
    G.close()


# the degree order and both directions of a build: id ranges around the parts of the
# degree count, a vertex with most of the arcs, no arcs, one arc, undirected
@pytest.mark.parametrize("n,m,und", [(2, 1, False), (1, 0, False), (257, 4000, False), (8193, 40000, True),
                                     (262145, 1500000, False), (2097151, 1200000, False), (2097153, 500000, True)])
def test_build_order_and_directions(dg, n, m, und):
    rng = np.random.default_rng(n)
    u = np.where(rng.random(2 * m + 8) < 0.4, n // 3, rng.integers(0, n, 2 * m + 8))
    v = rng.integers(0, n, 2 * m + 8)
    if n == 2:
        u, v = np.array([1]), np.array([0])
    if und:
        u, v = np.minimum(u, v), np.maximum(u, v)
    key = np.unique((u.astype(np.int64) << 32 | v)[u != v])
    key = rng.permutation(key)[:m]
    s, d = (key >> 32).astype(np.int32), (key & 0xFFFFFFFF).astype(np.int32)
    w = rng.integers(1, 100, s.size).astype(np.int32)
    G = dg.Graph(n, s, d, w, undirected=und)
    es, ed, ew = G.export()
    o = np.argsort(key)
    assert np.array_equal(es, s[o]) and np.array_equal(ed, d[o]) and np.array_equal(ew, w[o])
    # ranks read the reverse rows, the export the forward ones
    as_, ad = (np.concatenate([s, d]), np.concatenate([d, s])) if und else (s, d)
    want, _, _ = oracle.pagerank(n, as_, ad, 0.85, 1e-9, 1000)
    assert np.max(np.abs(G.pr_static(0.85, 1e-9, 1000)[0] - want)) <= 1e-10
    G.close()


# batches around the limit of the one-workgroup path, in every mode, over several batches
# (revivals, reused slots, repeats within a batch, deletions with re-insertions)
@pytest.mark.parametrize("und", [False, True])
@pytest.mark.parametrize("k", [1, 63, 65, 1023, 1025, 2047, 2048, 2049, 3071, 3072, 3073, 4095, 4096, 4097])
@pytest.mark.parametrize("diff_only", [0, 1])
def test_small_batch_sequences(dg, k, und, diff_only):
    rng = np.random.default_rng(7 * k + und)
    n = 3001
    if und:
        _, s, d = graphgen.rmat_undirected(12, 20000, 5)
    else:
        _, s, d, _ = graphgen.rmat_directed(12, 30000, 5)
    keep = (s < n) & (d < n)
    s, d = s[keep], d[keep]
    w = rng.integers(1, 100, s.size).astype(np.int32)
    c = dg.Config()
    c.diff_only = diff_only
    G = dg.Graph(n, s, d, w, undirected=und, config=c)
    q = G.tc_attach() if und else G.sssp_attach(0)
    for step in range(4):
        # half existing edges, half random pairs, some of them repeated, random ops
        i = rng.integers(0, s.size, k)
        a, b = rng.integers(0, n, k), rng.integers(0, n, k)
        old = rng.random(k) < 0.5
        bs, bd = np.where(old, s[i], a), np.where(old, d[i], b)
        rep = rng.integers(0, k, k)
        again = rng.random(k) < 0.1
        bs, bd = np.where(again, bs[rep], bs), np.where(again, bd[rep], bd)
        bd = np.where(bs == bd, (bd + 1) % n, bd)
        op = rng.integers(0, 2, k)
        bw = rng.integers(1, 100, k)
        if und:  # weights of an undirected pair are not part of the comparison
            bw[:] = 1
        batch = (bs.astype(np.int32), bd.astype(np.int32), bw.astype(np.int32), op.astype(np.uint8))
        G.apply(*batch)
        s, d, w, _ = oracle.apply(n, s, d, w, *batch, undirected=und)
        es, ed, ew = G.export()
        o = np.argsort(s.astype(np.int64) << 32 | d)
        assert np.array_equal(es, s[o]) and np.array_equal(ed, d[o])
        if und:
            assert q.read() == oracle.triangles(n, s, d)
        else:
            assert np.array_equal(ew, w[o])
            assert np.array_equal(q.read()[0], oracle.sssp(n, s, d, w, 0))
    G.close()


# one-workgroup end of a rank step: sizes around its threads and its limits, plain and
# extrapolated steps, rows over several tiles, dangling vertices
@pytest.mark.parametrize("extrap", [0, 1])
@pytest.mark.parametrize("n", [3, 1023, 1025, 4096, 4097, 32767, 32768, 32769])
def test_rank_step_end(dg, n, extrap):
    rng = np.random.default_rng(n)
    m = min(6 * n, n * (n - 1) // 2)
    u, v = (n * rng.random(4 * m) ** 2).astype(np.int64), rng.integers(0, n, 4 * m)
    v = np.where(rng.random(4 * m) < 0.15, n // 2, v)  # one row of many entries
    key = rng.permutation(np.unique((u << 32 | v)[u != v]))[:m]
    s, d = (key >> 32).astype(np.int32), (key & 0xFFFFFFFF).astype(np.int32)
    c = dg.Config()
    c.pr_extrapolate = extrap
    G = dg.Graph(n, s, d, None, config=c)
    q = G.pr_attach(0.85, 1e-9, 1000)
    for step in range(3):
        want, _, _ = oracle.pagerank(n, s, d, 0.85, 1e-9, 1000)
        rank, _, conv = q.read()
        assert conv and np.max(np.abs(rank - want)) <= 1e-10
        if n > 100:
            b = graphgen.update_batch(n, s, d, n // 20, step)
            G.apply(*b)
            s, d, _, _ = oracle.apply(n, s, d, np.ones(s.size, np.int32), *b)
    G.close()


# ranks of odd and even vertex counts on both sides of the tiles' arcs-per-vertex line and
# of the apply's streaming line.  Each side stops at an L1 step of tol, which leaves it
# within tol d / (1 - d) of the fixed point.
@pytest.mark.parametrize("n,deg", [(40000, 4), (40001, 4), (40001, 12), ((1 << 23) - 1, 0.1), ((1 << 23) + 1, 0.1)])
def test_rank_vectors(dg, n, deg):
    rng = np.random.default_rng(n)
    key = np.unique(rng.integers(0, n, int(n * deg)) << 32 | (n * rng.random(int(n * deg)) ** 2).astype(np.int64))
    key = key[(key >> 32) != (key & 0xFFFFFFFF)]
    s, d = (key >> 32).astype(np.int32), (key & 0xFFFFFFFF).astype(np.int32)
    G = dg.Graph(n, s, d, None)
    q = G.pr_attach(0.85, 1e-9, 1000)
    for step in range(2):
        want, _, _ = oracle.pagerank(n, s, d, 0.85, 1e-9, 1000)
        rank, _, conv = q.read()
        assert conv and np.sum(np.abs(rank - want)) <= 2 * 1e-9 * 0.85 / 0.15
        b = graphgen.update_batch(n, s, d, 5000, step)
        G.apply(*b)
        s, d, _, _ = oracle.apply(n, s, d, np.ones(s.size, np.int32), *b)
    G.close()


# static triangle count on the rows' beginnings (degree order as built) and on built lists
# (after batches changed the degrees), with forward lists around the group sizes, ids on
# both sides of the bitmap's 32,768 and lists long enough to be searched
@pytest.mark.parametrize("n,core,m", [(3, 3, 0), (300, 65, 200), (2000, 130, 3000), (40000, 513, 60000), (70000, 1100, 120000)])
def test_static_count_lists(dg, n, core, m):
    rng = np.random.default_rng(n)
    ids = rng.permutation(n)
    a, b = np.triu_indices(core, 1)
    keep = rng.random(a.size) < 0.9
    u = np.concatenate([ids[a[keep]], rng.integers(0, n, m), ids[rng.integers(0, core, m)]])
    v = np.concatenate([ids[b[keep]], rng.integers(0, n, m), rng.integers(0, n, m)])
    far = ids[-200:] if n > 40000 else ids[:0]  # a second clique of low degree: ids past the bitmap
    fa, fb = np.triu_indices(far.size, 1)
    pick = rng.random(fa.size) < 0.05
    u, v = np.concatenate([u, far[fa[pick]]]), np.concatenate([v, far[fb[pick]]])
    key = np.unique((np.minimum(u, v) << 32 | np.maximum(u, v))[u != v])
    s, d = (key >> 32).astype(np.int32), (key & 0xFFFFFFFF).astype(np.int32)
    G = dg.Graph(n, s, d, None, undirected=True)
    assert G.tc_static() == oracle.triangles(n, s, d)
    if n > 3:
        batch = graphgen.update_batch(n, s, d, max(40, m // 20), 1)
        G.apply(*batch)
        s, d, _, _ = oracle.apply(n, s, d, np.ones(s.size, np.int32), *batch, undirected=True)
        assert G.tc_static() == oracle.triangles(n, s, d)
    G.close()


# triangles of changed edges between rows whose lengths lie around the steps of the search
# (groups of four, the fenced length, pieces of 64 and 256), before and after the longer row
# holds tombstones, marks and diff-level entries at its ends
@pytest.mark.parametrize("long", [1, 3, 4, 5, 127, 129, 1025, 20000])
@pytest.mark.parametrize("short", [1, 64, 65, 257])
def test_changed_edge_rows(dg, long, short):
    rng = np.random.default_rng(1000 * short + long)
    n = 30000
    hub, low = 15000, 20000  # the two ends of every changed edge
    nb = np.sort(rng.choice(np.setdiff1d(np.arange(n), [hub, low]), max(long, short) + 40, replace=False))
    a = nb[:long] if long < nb.size else nb
    b = np.unique(rng.choice(nb, short, replace=False))
    s = np.concatenate([np.full(a.size, hub), np.full(b.size, low)]).astype(np.int32)
    d = np.concatenate([a, b]).astype(np.int32)
    u, v = np.minimum(s, d), np.maximum(s, d)
    G = dg.Graph(n, u, v, None, undirected=True)
    q = G.tc_attach()
    for step in range(4):
        # the edge itself appears and goes; the rows' ends go, and come back as new entries
        bs, bd, op = [hub], [low], [1 - step % 2]
        ends = [a[0], a[-1], b[0], b[-1]]
        if step in (1, 2):
            for x, r in ((ends[0], hub), (ends[1], hub), (ends[2], low), (ends[3], low)):
                bs.append(r), bd.append(x), op.append(step - 1)
        if step == 3:
            far = np.setdiff1d(np.arange(10), np.concatenate([a, b]))[:2]
            for x in far:
                bs += [hub, low]
                bd += [x, x]
                op += [1, 1]
        batch = (np.array(bs, np.int32), np.array(bd, np.int32), np.ones(len(bs), np.int32), np.array(op, np.uint8))
        G.apply(*batch)
        u, v, _, _ = oracle.apply(n, u, v, np.ones(u.size, np.int32), *batch, undirected=True)
        assert q.read() == oracle.triangles(n, u, v), step
    G.close()


# changed edges finished by windows of 16, rows on both sides of the 32 candidates
@pytest.mark.parametrize("k", [1, 15, 16, 17, 65, 400])
@pytest.mark.parametrize("density", [0.15, 0.4, 0.7])
def test_changed_edges_of_short_rows(dg, k, density):
    rng = np.random.default_rng(k)
    n = 80
    a, b = np.triu_indices(n, 1)
    keep = rng.random(a.size) < density * rng.random(n)[a] * 1.5
    s, d = a[keep].astype(np.int32), b[keep].astype(np.int32)
    G = dg.Graph(n, s, d, None, undirected=True)
    q = G.tc_attach()
    for step in range(3):
        batch = graphgen.update_batch(n, s, d, min(k, s.size), step, undirected=True)
        G.apply(*batch)
        s, d, _, _ = oracle.apply(n, s, d, np.ones(s.size, np.int32), *batch, undirected=True)
        assert q.read() == oracle.triangles(n, s, d), step
    G.close()


# the same step ends with diff levels around the entries that one workgroup takes
@pytest.mark.parametrize("k", [3500, 4500])
def test_rank_step_end_diff_entries(dg, k):
    rng = np.random.default_rng(k)
    n = 3000
    key = rng.permutation(n * n)[: 12000 + k]
    key = key[key // n != key % n]
    s, d = (key // n).astype(np.int32), (key % n).astype(np.int32)
    c = dg.Config()
    c.merge_threshold, c.diff_only = 10.0, 1
    G = dg.Graph(n, s[k:], d[k:], None, config=c)
    q = G.pr_attach(0.85, 1e-9, 1000)
    G.apply(s[:k], d[:k], np.ones(k, np.int32), np.ones(k, np.uint8))
    want, _, _ = oracle.pagerank(n, s, d, 0.85, 1e-9, 1000)
    rank, _, conv = q.read()
    assert conv and np.max(np.abs(rank - want)) <= 1e-10
    G.close()
