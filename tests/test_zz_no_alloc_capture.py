"""ccm_dev_noalloc under graph capture: every replay gives the eager result for
the series then in the buffers, with other host allocations, calls of the
context and device work between the replays.
"""
import numpy as np
import pytest

from paper_1905_00565_amd import capi, synth


@pytest.mark.gpu
def test_captured_call_replays():
    torch = pytest.importorskip("torch")
    N, E, tau, L, r = 500, 3, 1, [60, 300, 498], 20
    pairs = [synth.coupled_logistic(N, x0, 0.2) for x0 in (0.4, 0.55, 0.7, 0.85)]
    X, Y = (torch.zeros(N, dtype=torch.float64, device="cuda") for _ in range(2))
    a = torch.zeros(len(L), r, dtype=torch.float64, device="cuda")
    b = torch.zeros_like(a)
    with capi.Context(0) as ctx:
        side = torch.cuda.Stream()

        def call(out, stream):
            ctx.ccm_dev_noalloc(X, Y, E, tau, L, r, 3, *out, stream=stream)

        def load(k):
            for d, v in zip((X, Y), pairs[k]):
                d.copy_(torch.tensor(v))
            torch.cuda.synchronize()

        load(0)
        with torch.cuda.stream(side):
            call((a, b), side)                      # once before the capture
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            call((a, b), torch.cuda.current_stream())
        for k in (1, 2, 3, 1):
            load(k)
            want = [torch.zeros_like(a) for _ in range(2)]
            call(want, torch.cuda.current_stream())
            torch.cuda.synchronize()
            junk = [np.full(30_000, 7 * k, dtype=np.uint8) for _ in range(200)]
            ctx.ccm(*pairs[0], 2, 1, [100], 3, 1)
            a.fill_(-7.0), b.fill_(-7.0)
            graph.replay()
            torch.cuda.synchronize()
            del junk
            assert torch.equal(a, want[0]) and torch.equal(b, want[1]), k
