"""The kernels that only some calls reach, against the unbatched scan
(CCM_FLAG_PLAIN), bit for bit.  test_plan.py asserts on the CPU that the planner
sends each of these cases to its kernel.
"""
import numpy as np
import pytest

from paper_1905_00565_amd import capi, synth

pytestmark = pytest.mark.gpu

# Queries per lane of the scan: a spread launch gives 64 queries to a
# wavefront, 64 Q to a run, 256 Q to a tile.
Q = {1: 3, 2: 4, 3: 4, 4: 4, 5: 3, 6: 2, 8: 2, 10: 2}

# (E, tau, embedded points, L, exclusion_radius, query_set): the last wavefront,
# run and tile hold one query, are full, or miss one; the libraries are the
# whole embedding and a small one, with library-point queries sizes around 64
SPREAD = [(E, tau, ne, L, excl, 0)
          for E, tau in ((1, 1), (2, 3), (3, 1), (5, 2), (6, 1), (10, 1))
          for ne, excl in ((64 * (256 // 64) + 1, 0), (64 * Q[E] * 4 - 1, 3), (64 * Q[E] * 4, 0),
                           (64 * Q[E] * 4 + 1, 0), (64 * Q[E] * 5 + 64, 0))
          for L in ([20 + E, ne],)]
SPREAD += [(E, 1, 64 * Q[E] * 4 + 30, [63, 64, 65, 64 * Q[E] - 1, 64 * Q[E] + 1, 64 * Q[E] * 4 + 1],
            excl, 1) for E in (1, 3, 5, 8) for excl in (0, 5)]

# (M, N, E, tau, L, r, exclusion_radius): one target column, two and the last of
# 64, more than 64, M odd and even; groups whose last sixteen libraries and
# last four are partial
GROUPED = [
    (70, 2500, 2, 1, [1200, 2400], 35, 0),
    (67, 2300, 7, 1, [1100, 2200], 40, 0),
    (65, 1700, 10, 1, [900, 1600], 45, 0),
    (63, 3001, 3, 2, [900, 1500, 2990], 35, 4),
    (34, 9001, 5, 1, [4000, 8000], 40, 0),
    (51, 4100, 1, 1, [1500, 2100], 49, -1),
]


@pytest.fixture(scope="module")
def ctx():
    c = capi.Context(0)
    yield c
    c.close()


def same(a, b):
    return np.array_equal(a.view(np.uint64), b.view(np.uint64))


@pytest.mark.parametrize("case", SPREAD, ids=[str(c) for c in SPREAD])
def test_spread_edges(ctx, case):
    E, tau, ne, L, excl, qs = case
    N = ne + (E - 1) * tau
    X, Y = synth.coupled_logistic(N)
    if E % 2:
        rng = np.random.default_rng(N)
        X, Y = synth.quantised_series(N, 5, rng), synth.quantised_series(N, 7, rng)
    kw = dict(exclusion_radius=excl, query_set=qs)
    a = ctx.ccm_sweep(X, Y, [E], [tau], L, 4, 9, **kw)
    b = ctx.ccm_sweep(X, Y, [E], [tau], L, 4, 9, flags=capi.CCM_FLAG_PLAIN, **kw)
    assert same(a, b)


@pytest.mark.parametrize("case", GROUPED, ids=[str(c) for c in GROUPED])
def test_grouped_targets(ctx, case):
    M, N, E, tau, L, r, excl = case
    S, _ = synth.logistic_network(M, N, seed=M)
    a = ctx.ccm_matrix(S, E, tau, L, r, 3, exclusion_radius=excl)
    b = ctx.ccm_matrix(S, E, tau, L, r, 3, exclusion_radius=excl, flags=capi.CCM_FLAG_PLAIN)
    assert same(a, b)
