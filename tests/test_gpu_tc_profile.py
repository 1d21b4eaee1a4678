"""The bytes that the profile gives the two launches of a triangle delta are those each
launch moves: row bounds, entries of the shorter row and search steps into the longer."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import paper_2507_11094_amd as m
    return m


def profiled(dg, G, *batch):
    dg.dg_profile_reset()
    dg.dg_profile_enable(True)
    try:
        G.apply(*batch)
        return {k: v["bytes"] for k, v in dg.dg_profile_read().items() if k.startswith("tc_")}
    finally:
        dg.dg_profile_enable(False)
        dg.dg_profile_reset()


def test_short_edges(dg):
    n, m = 50000, 100000  # rows of at most 32 entries: the first launch finishes every edge
    rng = np.random.default_rng(4)
    u, v = rng.integers(0, n, m), rng.integers(0, n, m)
    key = np.unique((np.minimum(u, v) << 32 | np.maximum(u, v))[u != v])
    s, d = (key >> 32).astype(np.int32), (key & 0xFFFFFFFF).astype(np.int32)
    deg = np.bincount(s, minlength=n) + np.bincount(d, minlength=n)
    assert deg.max() <= 32
    G = dg.Graph(n, s, d, None, undirected=True)
    G.tc_attach()
    gone = rng.permutation(s.size)[:7001]
    a, b = deg[s[gone]], deg[d[gone]]
    short, long = np.minimum(a, b), np.maximum(a, b)
    steps = np.array([int(x).bit_length() for x in long])
    got = profiled(dg, G, s[gone], d[gone], None, np.zeros(gone.size, np.uint8))
    G.close()
    assert got == {"tc_items": 4.0 * (8 * gone.size + short.sum() + (short * steps).sum()), "tc_delta": 0.0}


def test_long_edge(dg):
    n = 100  # complete: rows of 99 entries, one work item for the one edge
    s, d = (x.astype(np.int32) for x in np.triu_indices(n, 1))
    G = dg.Graph(n, s, d, None, undirected=True)
    G.tc_attach()
    got = profiled(dg, G, s[:1], d[:1], None, np.zeros(1, np.uint8))
    G.close()
    assert got == {"tc_items": 32.0, "tc_delta": 4.0 * (8 + 99 + 99 * 7)}
