"""The degree order of a build over the plans of the degree count (one and two passes of
parting, parts of one and of several LDS ranges, few and many copies): among parents of
equal distance the library keeps the one that stands first in its order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per", [1, 40])
@pytest.mark.parametrize("n", [300, 8192, 8193, (1 << 21) + 1, 1 << 24, (1 << 24) + 1, (1 << 25) + 3, (1 << 26) + 1])
def test_first_of_equal_parents(n, per):
    import paper_2507_11094_amd as dg

    rng = np.random.default_rng(n + per)
    a = min(n // 4, 20000)
    ids = np.unique(np.concatenate([[1, n - 1, n // 2], rng.integers(1, n, 4 * a)]))
    ids = rng.permutation(ids)
    mid, end = ids[: ids.size // 2], ids[ids.size // 2:]
    # 0 -> every mid; every mid -> some ends, a few mids -> many
    deg = np.minimum(1 + (per * rng.pareto(1.5, mid.size)).astype(np.int64), end.size // 2)
    s2 = np.repeat(mid, deg)
    d2 = end[rng.integers(0, end.size, s2.size)]
    key = np.unique(s2 << 32 | d2)
    key = rng.permutation(np.concatenate([mid, key]))  # (0 << 32 | mid: the arcs of vertex 0)
    s, d = (key >> 32).astype(np.int32), (key & 0xFFFFFFFF).astype(np.int32)
    G = dg.Graph(n, s, d, None)
    dist, parent = G.sssp_attach(0).read()
    G.close()
    u, c = np.unique(s, return_counts=True)
    at = np.searchsorted(u, s)
    # the place of an arc's tail in the order: degree falling, then id
    place = (c.max() - c[at]).astype(np.int64) << 32 | s
    two = s != 0
    first = np.full(end.size, np.iinfo(np.int64).max)
    order = np.argsort(end)
    np.minimum.at(first, order[np.searchsorted(end[order], d[two])], place[two])
    hit = first != np.iinfo(np.int64).max
    assert np.array_equal(dist[end[hit]], np.full(hit.sum(), 2))
    assert np.array_equal(parent[end[hit]], (first[hit] & 0xFFFFFFFF).astype(np.int32))
    assert np.all(parent[mid] == 0)
