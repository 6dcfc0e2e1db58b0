"""Visiting orders: sorted in chunks of 4096 or 1024 keys and merged, then split level
by level along a k-d tree.  Every point must be visited exactly once at chunk
and node edges and among tied keys: a point lost or taken twice moves rho by
about 1/N (1e-5 and more here), while the GPU's and the oracle's sums, both in
binary64, differ by rounding only (some N 2^-53 < 1e-11).
"""
import numpy as np
import pytest

import oracle
from paper_1905_00565_amd import capi, synth

pytestmark = pytest.mark.gpu

# (N, E, tau, series): one chunk and its edges, two to 17 chunks with short
# last ones; E = 1 by value, 2 by Hilbert position, 3 and up by k-d levels
CASES = [(n, E, tau, kind)
         for n in (24, 97, 2049, 4096, 4097, 8193, 12289, 16385)
         for E, tau in ((1, 1), (2, 3), (3, 1), (7, 2))
         for kind in ("logistic", "quantised")
         if n - (E - 1) * tau >= E + 3]


@pytest.fixture(scope="module")
def ctx():
    c = capi.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_every_point_once(ctx, case):
    N, E, tau, kind = case
    X, Y = synth.coupled_logistic(N)
    if kind == "quantised":
        rng = np.random.default_rng(N)
        X, Y = synth.quantised_series(N, 5, rng), synth.quantised_series(N, 7, rng)
    L = [min(N - (E - 1) * tau, E + 40)]
    oracle.build(force=False)
    got = ctx.ccm(X, Y, E, tau, L, 2, 3)
    want = oracle.default().ccm(X, Y, E, tau, L, 2, 3)
    for g, w in zip(got[:2], want[:2]):
        g, w = np.asarray(g), np.asarray(w)
        assert np.array_equal(np.isnan(g), np.isnan(w))
        assert np.allclose(g, w, rtol=0, atol=1e-9, equal_nan=True)
