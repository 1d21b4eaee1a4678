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
