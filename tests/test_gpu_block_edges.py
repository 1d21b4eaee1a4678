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
