"""NaN in a device series.  The device-pointer forms do not read their series
on the host, so a NaN there is not refused.  It must stay where it is: the
direction that searches the series' manifold has no skill (NaN), and the other
direction, whose targets here lie past the NaN, is the clean call's bit for bit.

The NaN stand before the first target time (E-1) tau.  E >= 3: k-d visiting
orders.  Scanned and walked realizations, every series in both roles.
"""
import numpy as np
import pytest

from paper_1905_00565_amd import capi, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx():
    c = capi.Context(0)
    yield c
    c.close()


def same(a, b):
    return torch.equal(a.view(torch.int64), b.view(torch.int64))


# (N, E, tau, how many NaN, L, r, flags): one NaN; more than fit a bin's 256
# or 1024 ranked keys; a node of NaN alone; calls that scan, spread and walk
CASES = [
    (4000, 3, 1, 1, [40, 900], 3, 0),
    (4000, 3, 1, 1, [900, 3998], 70, 0),
    (777, 3, 2, 4, [51, 203, 770], 33, 0),
    (5000, 10, 30, 270, [100, 4000], 3, 0),
    (5000, 10, 30, 270, [1000, 4000], 70, 0),
    (6000, 4, 500, 1400, [2000, 4400], 40, capi.CCM_FLAG_TABLE),
    (3000, 5, 7, 28, [500, 2900], 40, capi.CCM_FLAG_NO_GRAPH),
    (3000, 5, 7, 28, [500, 2900], 90, capi.CCM_FLAG_NESTED),
]


@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_nan_stays_in_its_series(ctx, case):
    N, E, tau, bad, L, r, flags = case
    X, Y = (torch.tensor(v, device="cuda") for v in synth.coupled_logistic(N))
    clean = torch.empty(2, len(L), r, dtype=torch.float64, device="cuda")
    ctx.ccm_sweep_dev(X, Y, [E], [tau], L, r, 5, clean, flags=flags)
    torch.cuda.synchronize()
    for which in (0, 1):
        s = [X.clone(), Y.clone()]
        s[which][(E - 1) * tau - bad:(E - 1) * tau] = float("nan")
        for _ in range(2):
            got = torch.full_like(clean, -7.0)
            ctx.ccm_sweep_dev(*s, [E], [tau], L, r, 5, got, flags=flags)
            torch.cuda.synchronize()
            # rho[0]: X predicted from Y's manifold; rho[1]: Y from X's
            assert same(got[which], clean[which])
            assert torch.isnan(got[1 - which]).all()


def test_nan_noalloc(ctx):
    N, E, tau, L, r = 777, 3, 2, [51, 203, 770], 33
    X, Y = (torch.tensor(v, device="cuda") for v in synth.coupled_logistic(N))
    st = torch.cuda.current_stream()
    out = []
    for bad in (0, 4):
        X[4 - bad:4] = float("nan")
        a = torch.full((len(L), r), -7.0, dtype=torch.float64, device="cuda")
        b = torch.full_like(a, -7.0)
        ctx.ccm_dev_noalloc(X, Y, E, tau, L, r, 5, a, b, stream=st)
        torch.cuda.synchronize()
        out.append((a, b))
    assert same(out[0][0], out[1][0])
    assert torch.isnan(out[1][1]).all()


def test_nan_matrix_walked(ctx):
    """The causal matrix through neighbour rows."""
    M, N, E, tau, L, r = 5, 1500, 4, 2, [900, 1490], 12
    S = torch.tensor(synth.logistic_network(M, N, seed=5)[0], device="cuda")
    kw = dict(flags=capi.CCM_FLAG_TABLE)
    ctx.profile_enable(True)
    ctx.profile_read(reset=True)
    clean = torch.empty(M, M, len(L), r, dtype=torch.float64, device="cuda")
    ctx.ccm_matrix_dev(S, E, tau, L, r, 3, clean, **kw)
    torch.cuda.synchronize()
    walked = ctx.profile_read(reset=True)["table_realizations"]
    ctx.profile_enable(False)
    assert walked == M * (M - 1) * len(L) * r
    S[2, 1:6] = float("nan")
    got = torch.full_like(clean, -7.0)
    ctx.ccm_matrix_dev(S, E, tau, L, r, 3, got, **kw)
    torch.cuda.synchronize()
    keep = [a for a in range(M) if a != 2]
    assert same(got[keep].contiguous(), clean[keep].contiguous())
    assert torch.isnan(got[2]).all()
