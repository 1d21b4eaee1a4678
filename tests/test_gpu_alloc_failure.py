"""A graph that cannot be built for want of device memory gives back all it had taken."""
import gc

import numpy as np
import pytest

import graphgen
import paper_2507_11094_amd as dg

pytestmark = pytest.mark.gpu


class FailingHook(dg.TorchAllocatorHook):
    def __init__(self):
        self.left = 0  # allocations that still succeed
        super().__init__()

    def _alloc(self, nbytes, ctx):
        if self.left == 0:
            return None
        self.left -= 1
        return super()._alloc(nbytes, ctx)


@pytest.mark.parametrize("und", [False, True])
def test_failed_builds_keep_nothing(und):
    import ctypes

    gc.collect()  # graphs of earlier tests must be gone before the allocator changes
    if und:
        n, s, d = graphgen.rmat_undirected(10, 8 << 10, 3)
    else:
        n, s, d, _ = graphgen.rmat_directed(10, 8 << 10, 3)
    hook = FailingHook()
    dg._check(dg.load_library().dg_set_allocator(ctypes.cast(hook.c_alloc, ctypes.c_void_p),
                                                 ctypes.cast(hook.c_free, ctypes.c_void_p), None))
    try:
        for k in range(200):
            hook.left = k
            try:
                G = dg.Graph(n, s, d, np.ones(s.size, np.int32), undirected=und)
            except dg.DGError:
                assert hook.live_bytes() == 0, f"{k} allocations"
                continue
            G.close()
            assert hook.live_bytes() == 0
            break
        else:
            pytest.fail("no build within 200 allocations")
    finally:
        dg.use_default_allocator()
