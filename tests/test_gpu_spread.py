"""Launches of few items take 64 queries per wavefront and form the moments
apart; the plain form scans a tile per workgroup.  Same neighbours, same
operations, same merge order: rho must agree bit for bit at tile and run
edges, with ties, exclusions and library-point queries.
"""
import numpy as np
import pytest

from paper_1905_00565_amd import capi, synth

pytestmark = pytest.mark.gpu

CASES = [(N, E, tau, excl, qs)
         for N in (40, 127, 300, 1023, 1100, 2500)
         for E, tau in ((1, 1), (2, 2), (3, 1), (5, 1), (6, 1), (8, 2), (10, 1))
         for excl, qs in ((0, 0), (-1, 1), (4, 0))
         if N - (E - 1) * tau > 30]


@pytest.fixture(scope="module")
def ctx():
    c = capi.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_spread_equals_plain(ctx, case):
    N, E, tau, excl, qs = case
    X, Y = synth.coupled_logistic(N)
    if N % 2:
        rng = np.random.default_rng(N)
        X, Y = synth.quantised_series(N, 5, rng), synth.quantised_series(N, 7, rng)
    ne = N - (E - 1) * tau
    L = [min(ne, 25), ne // 2 + 12, ne]
    kw = dict(exclusion_radius=excl, query_set=qs)
    a = ctx.ccm_sweep(X, Y, [E], [tau], L, 5, 9, **kw)
    b = ctx.ccm_sweep(X, Y, [E], [tau], L, 5, 9, flags=capi.CCM_FLAG_PLAIN, **kw)
    assert np.array_equal(a.view(np.uint64), b.view(np.uint64))
