"""Memory kept from closed graphs goes back to the device while another graph is open."""
import gc

import numpy as np
import pytest

import graphgen
import oracle
import paper_2507_11094_amd as dg

pytestmark = pytest.mark.gpu


def test_release_beside_an_open_graph():
    import torch

    gc.collect()
    n, s, d, w = graphgen.rmat_directed(12, 16 << 12, graphgen.config_seed(0, 5))
    G = dg.Graph(n, s, d, w)
    q = G.sssp_attach(0)
    big = graphgen.rmat_directed(18, 16 << 18, graphgen.config_seed(0, 3))
    dg.release_memory()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    dg.Graph(*big).close()
    kept = before - torch.cuda.mem_get_info()[0]
    dg.release_memory()
    left = before - torch.cuda.mem_get_info()[0]
    assert kept > 0 and left < kept / 4
    b = graphgen.update_batch(n, s, d, 700, 9)
    G.apply(*b)
    s, d, w, _ = oracle.apply(n, s, d, w, *b)
    assert np.array_equal(q.read()[0], oracle.sssp(n, s, d, w, 0))
    G.close()


def test_export_scratch_is_kept_for_the_next_export():
    import torch

    gc.collect()
    n, s, d, w = graphgen.rmat_directed(18, 16 << 18, graphgen.config_seed(0, 4))
    G = dg.Graph(n, s, d, w)
    dg.release_memory()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    first = G.export()
    assert before - torch.cuda.mem_get_info()[0] >= 3 * 4 * s.size  # rows, columns and weights
    second = G.export()
    assert all(np.array_equal(a, b) for a, b in zip(first, second))
    dg.release_memory()
    assert before - torch.cuda.mem_get_info()[0] < 4 * s.size
    G.close()
