"""Device memory kept between graphs: reuse with stale contents, give-back, threads."""
import gc
import threading

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import paper_2507_11094_amd as m
    return m


def check(dg, seed, scale=11, delta=0):
    n, s, d, w = graphgen.rmat_directed(scale, 16 << scale, graphgen.config_seed(0, seed))
    b = graphgen.update_batch(n, s, d, 500 + 37 * (seed % 11), seed)
    c = dg.Config()
    c.sssp_delta = delta
    G = dg.Graph(n, s, d, w, config=c)
    qs, qp = G.sssp_attach(0), G.pr_attach(0.85, 1e-9, 1000)
    G.apply(*b)
    s2, d2, w2, _ = oracle.apply(n, s, d, w, *b)
    ok = np.array_equal(qs.read()[0], oracle.sssp(n, s2, d2, w2, 0))
    ok &= bool(np.max(np.abs(qp.read()[0] - oracle.pagerank(n, s2, d2, 0.85, 1e-9, 1000)[0])) <= 1e-10)
    qs.detach()  # its memory may serve the graph of another thread from here on
    G.close()
    return ok


def test_graphs_on_reused_memory(dg):
    # sizes alternate, so that blocks are reused whole, in part and not at all
    for i, scale in enumerate([11, 11, 9, 11, 12, 9, 12, 11]):
        assert check(dg, 70 + i, scale, delta=40 * (i % 2))


def test_memory_is_given_back(dg):
    import torch

    gc.collect()  # graphs of earlier tests must be gone before the allocator changes
    dg.use_default_allocator()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    n, s, d, w = graphgen.rmat_directed(18, 16 << 18, graphgen.config_seed(0, 3))
    dg.Graph(n, s, d, w).close()
    kept = before - torch.cuda.mem_get_info()[0]
    dg.use_default_allocator()
    left = before - torch.cuda.mem_get_info()[0]
    assert kept > 0 and left < kept / 4


def test_threads_share_the_memory(dg):
    bad = []

    def work(t):
        for i in range(4):
            if not check(dg, 100 + 10 * t + i, 9 + (t + i) % 3):
                bad.append((t, i))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for x in threads:
        x.start()
    for x in threads:
        x.join()
    assert not bad
