"""One-workgroup batches filled to their limit (3,072 arcs) with insertions or deletions
alone, directed and undirected, against the oracle: the third key per lane of the sort,
the third round of every loop, revivals, hole reuse and the reverse keys past 2,048."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import paper_2507_11094_amd as m
    return m


def pairs(rng, n, k, und, have=()):
    """k distinct pairs (u < v if undirected) that are not in `have`."""
    key = np.zeros(0, np.int64)
    while key.size < k:
        u, v = rng.integers(0, n, 2 * k + 64), rng.integers(0, n, 2 * k + 64)
        if und:
            u, v = np.minimum(u, v), np.maximum(u, v)
        new = (u << 32 | v)[u != v]
        key = np.unique(np.concatenate([key, new[~np.isin(new, have)]]))
    return rng.permutation(key)[:k]


def split(key):
    return (key >> 32).astype(np.int32), (key & 0xFFFFFFFF).astype(np.int32)


# updates: directed ones are one arc each, undirected two, so 1,536 is the last undirected
# batch of one workgroup and 3,072 the last directed one
@pytest.mark.parametrize("k,und", [(1024, True), (1025, True), (1535, True), (1536, True), (1537, True),
                                   (2047, False), (2049, False), (3071, False), (3072, False), (3073, False)])
@pytest.mark.parametrize("diff_only", [0, 1])
@pytest.mark.parametrize("merge", [0.05, 10.0])
def test_one_kind_of_update(dg, k, und, diff_only, merge):
    rng = np.random.default_rng(k + diff_only)
    n = 2500
    key = pairs(rng, n, 12000, und)
    s, d = split(key)
    w = np.ones(s.size, np.int32) if und else rng.integers(1, 100, s.size).astype(np.int32)
    c = dg.Config()
    c.diff_only, c.merge_threshold = diff_only, merge
    G = dg.Graph(n, s, d, w, undirected=und, config=c)
    q = G.tc_attach() if und else G.sssp_attach(0)
    fresh = pairs(rng, n, 3 * k, und, key)
    gone = rng.permutation(key)
    steps = [(fresh[:k], 1),              # new keys only
             (gone[:k], 0),               # deletions only
             (fresh[k:2 * k], 1),         # new keys beside the holes they leave
             (gone[:k], 1),               # the deleted arcs again: revivals, or new where the hole is taken
             (np.concatenate([fresh[:k // 2], gone[k:k + k - k // 2]]), 0),
             (fresh[2 * k:], 1)]
    for arcs, op in steps:
        bs, bd = split(rng.permutation(arcs))
        bw = np.ones(k, np.int32) if und else rng.integers(1, 100, k).astype(np.int32)
        batch = (bs, bd, bw, np.full(k, op, np.uint8))
        st = G.apply(*batch)
        assert (st.deleted, st.inserted) == ((0, k) if op else (k, 0))
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
