"""Kernels that every call runs use no scratch memory.  The runtime takes a
launch's scratch from the device by itself, and where nothing is left it ends
the process instead of returning an error.  Read from the metadata of the built
library's code object.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_1905_00565_amd import build, capi

LLVM = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.hipcc()))), "llvm", "bin")


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    if not os.path.exists(capi.LIBRARY):
        build.build_library()
    d = tmp_path_factory.mktemp("code")
    shutil.copy(capi.LIBRARY, d / "lib.so")
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", "lib.so"], cwd=d,
                   check=True, capture_output=True)
    sizes = {}
    for obj in os.listdir(d):
        if "gfx950" not in obj:
            continue
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", obj], cwd=d,
                               check=True, capture_output=True, text=True).stdout
        for k in re.split(r"\n  - \.", notes):
            name = re.search(r"\.symbol: +(\S+)", k)
            size = re.search(r"\.private_segment_fixed_size: +(\d+)", k)
            if name and size:
                sizes[name.group(1)] = int(size.group(1))
    return sizes


@pytest.mark.parametrize("kernel", ["k_ingest", "k_embed", "k_series_range", "k_sort_chunks",
                                    "k_merge_runs", "k_kd_level", "k_query_order", "k_sample",
                                    "k_gather", "k_finalize"])
def test_no_scratch(scratch, kernel):
    found = {n: s for n, s in scratch.items() if f"{len(kernel)}{kernel}" in n}
    assert found and all(s == 0 for s in found.values()), found
