"""The planner (host code of libccm): which realizations of a call walk
neighbour rows, and what memory that takes.  Runs without a GPU: a small
program (tests/native/plan_report.cpp) linked with the library prints the plan.
"""
import json
import os
import subprocess

import pytest

import test_gpu_paths as paths
import test_gpu_rows as rows
import test_gpu_rows_uneven as uneven
from paper_1905_00565_amd import build, capi

HERE = os.path.dirname(os.path.abspath(__file__))
GIB = 1 << 30


@pytest.fixture(scope="session")
def plan(tmp_path_factory):
    if not os.path.exists(capi.LIBRARY):
        build.build_library()
    exe = str(tmp_path_factory.mktemp("plan") / "plan_report")
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(build.hipcc())))
    subprocess.run(
        ["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include",
         f"-I{build.INCLUDE}", f"-I{build.CSRC}", os.path.join(HERE, "native", "plan_report.cpp"),
         "-o", exe, capi.LIBRARY, f"-L{rocm}/lib", "-lamdhip64",
         f"-Wl,-rpath,{os.path.dirname(capi.LIBRARY)}", f"-Wl,-rpath,{rocm}/lib"], check=True)

    def report(N, E, tau, L, r, M=0, excl=0, query_set=0, flags=0, wave_limit=None, walk=1,
               spread=1, groups=(1 << 31) // 8 - 1):
        text = [",".join(str(x) for x in v) for v in (E, tau, L)]
        args = [M, N, *text, r, excl, query_set, flags]
        args += [8 * GIB if wave_limit is None else wave_limit, walk, spread, groups]
        out = subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True)
        return json.loads(out.stdout)

    return report


@pytest.mark.parametrize("kw", [
    dict(N=4_000_000, E=[1], tau=[1], L=[2_000_000, 4_000_000], r=64),
    dict(N=1_048_577, E=[1], tau=[1], L=[1_000_000], r=64),       # one past 64 libraries' output
    dict(N=1_000_000, E=[4], tau=[1], L=[500_000, 1_000_000], r=33, M=2),
    dict(N=4_000_000, E=[10], tau=[1], L=[4_000_000], r=6, M=2),
    dict(N=250_000, E=[1, 3], tau=[2], L=[100_000], r=64, flags=capi.CCM_FLAG_SHARED_E),
    dict(N=65_536, E=[2], tau=[1], L=[30_000, 65_000], r=64, flags=capi.CCM_FLAG_NESTED),
    dict(N=20_000, E=[4], tau=[1], L=[500, 5000, 20_000], r=40, M=64),
], ids=str)
def test_walk_memory_bound(plan, kw):
    """Neighbour rows and the walks' output stay within the stated 3.5 GiB, the
    output within its own bound."""
    p = plan(**kw)
    assert p["walked"] > 0
    assert p["out_bytes"] <= (GIB if kw.get("M") else GIB // 2)
    assert p["out_bytes"] + p["row_bytes"] <= 3.5 * GIB


NESTED, SHARED, TABLE = (capi.CCM_FLAG_NESTED, capi.CCM_FLAG_SHARED_E, capi.CCM_FLAG_TABLE)


@pytest.mark.parametrize("groups", [(1 << 31) // 8 - 1, 3, 0])
@pytest.mark.parametrize("kw", [
    dict(N=3000, E=[2, 5], tau=[1, 3], L=[100, 600, 3000], r=70),
    dict(N=3000, E=[2, 5], tau=[1], L=[100, 600, 3000], r=70, query_set=1, excl=3),
    dict(N=3000, E=[2, 5], tau=[1], L=[100, 600, 3000], r=70, wave_limit=4 << 20),
    dict(N=3000, E=[2, 5], tau=[1], L=[100, 600, 3000], r=70, flags=NESTED),
    dict(N=3000, E=[1, 3, 4], tau=[1, 2], L=[100, 600, 3000], r=70, flags=SHARED),
    dict(N=3000, E=[3], tau=[1], L=[100, 600, 3000], r=40, M=33),
    dict(N=900, E=[3], tau=[1], L=[100, 600], r=2, flags=TABLE),
    dict(N=900, E=[3], tau=[1], L=[100, 600], r=2),
], ids=str)
def test_every_tile_has_one_writer(plan, kw, groups):
    """Whatever part of a call walks, every tile of every result is formed once;
    also where the plan runs out of numbers for walk groups."""
    p = plan(**kw, groups=groups)
    assert p["missing"] == 0 and p["twice"] == 0
    assert p["groups"] <= groups


@pytest.mark.parametrize("N", [2048, 1_048_576, 1_048_577, 20_000_000])
def test_query_order_work(plan, N):
    """Placing an embedding's points in visiting order stays linear in the series."""
    assert plan(N=N, E=[2], tau=[3], L=[40], r=1)["order_reads"] <= 256 * N


# ---------------------------------------------------------------------------
# the GPU tests that compare two routes of a call take those two routes
# ---------------------------------------------------------------------------

def cases_of(test):
    return next(m.args[1] for m in test.pytestmark if m.name == "parametrize")


@pytest.mark.parametrize("case", paths.SPREAD, ids=str)
def test_spread_cases_spread(plan, case):
    E, tau, ne, L, excl, qs = case
    kw = dict(N=ne + (E - 1) * tau, E=[E], tau=[tau], L=L, r=4, excl=excl, query_set=qs)
    p = plan(**kw)
    assert p["spread_items"] == p["scan_items"] > 0 and p["walked"] == 0
    assert plan(**kw, flags=capi.CCM_FLAG_PLAIN, walk=0, spread=0)["spread_items"] == 0


@pytest.mark.parametrize("case", paths.GROUPED, ids=str)
def test_grouped_cases_group(plan, case):
    M, N, E, tau, L, r, excl = case
    p = plan(M=M, N=N, E=[E], tau=[tau], L=L, r=r, excl=excl)
    assert p["grouped_items"] >= 1024 and p["scan_items"] == 0
    assert p["missing"] == 0 and p["twice"] == 0


@pytest.mark.parametrize("excl,L", cases_of(uneven.test_uneven_rows_equal_scan))
def test_uneven_rows_are_long(plan, excl, L):
    p = plan(N=6 * 8192, E=[6], tau=[8192], L=L, r=64, excl=excl)
    assert p["row_width"] >= 768 and p["walked"] == 2 * 64 * len(L)


@pytest.mark.parametrize("excl,qs", cases_of(rows.test_rows_by_rule_equal_scan))
def test_rows_by_rule_cases_walk(plan, excl, qs):
    p = plan(N=3001, E=[2, 5, 10], tau=[1, 3], L=[40, 150, 600, 2000, 3001], r=70, excl=excl,
             query_set=qs)
    assert p["walked"] > 0 and p["scan_items"] > 0


@pytest.mark.parametrize("N,E,tau,L,r,excl,kind", cases_of(rows.test_nested_rows_equal_scan))
def test_nested_cases_take_both(plan, N, E, tau, L, r, excl, kind):
    kw = dict(N=N, E=[E], tau=[tau], L=L, excl=excl, flags=NESTED)
    assert plan(**kw, r=1)["walked"] == 0
    assert plan(**kw, r=r)["walked"] > 0


@pytest.mark.parametrize("N,Es,tau,L,r,excl,kind", cases_of(rows.test_shared_rows_equal_scan))
def test_shared_cases_take_both(plan, N, Es, tau, L, r, excl, kind):
    kw = dict(N=N, E=Es, tau=[tau], L=L, excl=excl, flags=SHARED)
    assert plan(**kw, r=1)["walked"] == 0
    assert plan(**kw, r=r)["walked"] > 0


def test_replayed_call_walks_and_scans(plan):
    p = plan(N=4000, E=[2, 5], tau=[1], L=[40, 1500, 3000], r=60)
    assert p["walked"] > 0 and p["scan_items"] > 0


# Shuffled series fill their embedding, and a row then costs a multiple of what it
# costs on an attractor.  Measured, ms walked / scanned / before there were rows.
@pytest.mark.parametrize("N,E,L,r,flags,walks", [
    (32768, 9, [200, 2048], 40, 0, False),       # 10.1 / 3.5 / 5.2
    (32768, 10, [200, 2048, 32768], 4, 0, False),   # 10.9 / 6.5 / 8.0
    (60000, 9, [200, 3750], 40, 0, False),       # 13.3 / 8.8 / 11.5
    (100000, 10, [200, 6250], 40, 0, False),     # 44.7 / 22.0 / 26.4
    (32768, 10, [200, 2048, 8192], 10, NESTED, False),   # 10.8 / 4.3 / 8.1
    (16000, 10, [500, 4000], 10, 0, True),       # 2.2 / 1.5 / 2.4
    (32768, 6, [500, 8192], 10, 0, True),        # 1.9 / 2.4 / 4.0
    (60000, 9, [500, 15000], 10, 0, True),       # 8.7 / 9.2 / 11.8
    (100000, 8, [200, 6250], 40, 0, True),       # 18.6 / 17.3 / 21.5
    (100000, 9, [200, 6250, 100000], 4, 0, True),   # 27.4 / 38.0 / 41.7
    (60000, 9, [200, 3750], 40, TABLE, True),    # asked for
])
def test_long_series_in_many_dimensions(plan, N, E, L, r, flags, walks):
    assert (plan(N=N, E=[E], tau=[1], L=L, r=r, flags=flags)["walked"] > 0) == walks


@pytest.mark.parametrize("kw,walked,width", [
    # 21.8 ms with rows of 1024 for the small libraries too, 10.7 with rows of 64
    (dict(M=70, N=17687, E=[1], tau=[2], L=[83, 164, 337, 551, 556, 11036, 11415, 11591, 14815],
          r=9), 70 * 4 * 9, 64),
    # 1.87 and 1.23
    (dict(N=5160, E=[8], tau=[1], L=[101, 185, 5160], r=11, excl=16), 2 * 11, 128),
    (dict(N=5003, E=[7], tau=[3], L=[101, 999, 3001, 4985], r=25, excl=10), 128, 192),
])
def test_library_point_queries_leave_small_libraries(plan, kw, walked, width):
    """A small library asks few of the rows that it would lengthen for all."""
    p = plan(**kw, query_set=1)
    assert (p["walked"], p["row_width"]) == (walked, width)
    assert p["missing"] == 0 and p["twice"] == 0


# ms walked / scanned / before there were rows
@pytest.mark.parametrize("M,N,E,tau,L,r,flags,walks", [
    (17, 2050, 5, 1, [30, 44, 48, 107, 374, 378, 397, 1377, 1730], 12, 0, False),  # 1.86 / 1.17 / 1.45
    (70, 9815, 8, 2, [45, 46, 54, 67, 82, 151, 292, 390, 1677, 9815], 4, 0, False),  # 34.1 / 25.0 / 25.7
    (33, 984, 1, 2, [23, 54, 92, 126, 205, 334, 595, 744, 984], 16, 0, False),   # 0.82 / 0.73 / 0.75
    (17, 9290, 7, 1, [31, 50, 75, 177, 1196, 2871, 3668], 11, 0, True),          # 5.1 / 6.1
    (64, 20000, 4, 1, [500, 2000, 20000], 10, 0, True),
    (8, 13797, 4, 2, [13797], 6, 0, True),                                       # few series
    (17, 2050, 5, 1, [30, 397, 1730], 12, TABLE, True),                          # asked for
])
def test_small_matrices_scan(plan, M, N, E, tau, L, r, flags, walks):
    p = plan(M=M, N=N, E=[E], tau=[tau], L=L, r=r, flags=flags)
    assert (p["walked"] > 0) == walks
    assert p["missing"] == 0 and p["twice"] == 0
