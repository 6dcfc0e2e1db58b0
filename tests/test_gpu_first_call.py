"""The first call of a plan with walks is issued directly, and its graph made
when it comes again (tests/native/first_call.cpp)."""
import os
import subprocess

import pytest

from paper_1905_00565_amd import build, capi

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.gpu
def test_no_graph_for_a_single_call(tmp_path):
    exe = str(tmp_path / "first_call")
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(build.hipcc())))
    subprocess.run(
        ["g++", "-O1", "-std=c++17", "-rdynamic", "-D__HIP_PLATFORM_AMD__",
         f"-I{rocm}/include", f"-I{build.INCLUDE}",
         os.path.join(HERE, "native", "first_call.cpp"), "-o", exe, capi.LIBRARY,
         f"-L{rocm}/lib", "-lamdhip64", "-ldl",
         f"-Wl,-rpath,{os.path.dirname(capi.LIBRARY)}", f"-Wl,-rpath,{rocm}/lib"], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout + out.stderr
