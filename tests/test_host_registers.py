"""Registers of the built kernels, read from the library's own code objects
(no GPU): limits that the kernels' occupancy, and so their measured times,
rest on."""

import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1711_11296_amd", "libsht.so")
LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled kernel name: (vector registers, spilled ones)}"""
    tools = [os.path.join(LLVM, t) for t in ("llvm-objdump", "llvm-readelf")]
    if not os.path.exists(LIB) or not all(os.path.exists(t) for t in tools):
        pytest.skip("needs the built library and ROCm's object tools")
    d = tmp_path_factory.mktemp("obj")
    shutil.copy(LIB, d)
    subprocess.run([tools[0], "--offloading", "libsht.so"], cwd=d, check=True, capture_output=True)
    out = {}
    for f in glob.glob(str(d / "*gfx950*")):
        notes = subprocess.run([tools[1], "--notes", f], check=True, capture_output=True, text=True).stdout
        for k in notes.split(".agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(_Z\S+)", k).group(1)
            out[name] = tuple(int(re.search(r"\.%s:\s+(\d+)" % w, k).group(1))
                              for w in ("vgpr_count", "vgpr_spill_count"))
    assert out
    return out


def _find(kernels, pattern):
    hits = [v for n, v in kernels.items() if re.search(pattern, n)]
    assert hits, pattern
    return hits


@pytest.mark.parametrize("ncb", [1, 2])
def test_generated_fp32_analysis_shares_a_unit_three_ways(kernels, ncb):
    """512 threads at 80 registers: three workgroups a compute unit (two above
    that measured 4-10 % slower)."""
    for vgpr, _ in _find(kernels, r"k_legendre_analysisIfLi%dELb1ELi[18]E" % ncb):
        assert vgpr <= 80
