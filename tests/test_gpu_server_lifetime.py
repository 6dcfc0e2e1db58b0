"""A server that is dropped without close() gives its memory back, and its
context lives as long as it does."""
import gc

import numpy as np
import pytest

from paper_1905_00565_amd import capi, synth


@pytest.mark.gpu
def test_dropped_server_frees_its_arena():
    torch = pytest.importorskip("torch")
    X, Y = synth.coupled_logistic(500)

    def free():
        gc.collect()
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    def server():
        # the context's only owner is the server
        return capi.Server(capi.Context(0), hbm_budget_bytes=1 << 30)

    server().close()                                # (one-time allocations)
    before = free()
    srv = server()
    gc.collect()
    t = srv.submit(X, Y, 2, 1, [100, 400], 3, 5)
    assert srv.wait(t) == capi.CCM_OK
    got = srv.result(t, 2, 3)[:2]
    assert before - free() > 1 << 29
    del srv
    assert before - free() < 1 << 29
    with capi.Context(0) as ctx:
        want = ctx.ccm(X, Y, 2, 1, [100, 400], 3, 5)[:2]
    assert all(np.array_equal(a, b) for a, b in zip(got, want))
