"""Whether a group of workgroups counts as being on one XCD, as host code: every wait ends, and only the right answer allows write-back stores."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def xcds(tmp_path_factory):
    clang = shutil.which("amdclang++") or "/opt/rocm/llvm/bin/clang++"
    if not os.path.exists(clang):
        pytest.skip("no clang++")
    out = str(tmp_path_factory.mktemp("xcds") / "xcds")
    subprocess.run([clang, "-x", "c++", "-std=c++20", "-pthread", "-O1", "-Wno-everything", "-I", os.path.join(HERE, "wave_on_cpu"), "-I", os.path.join(os.path.dirname(HERE), "paper_1904_04956_amd", "csrc"),
                    os.path.join(HERE, "wave_on_cpu", "xcds.cpp"), "-o", out], check=True)
    return lambda *what: subprocess.run([out, *what], capture_output=True, text=True, timeout=60, check=True).stdout.strip()


@pytest.mark.parametrize("what,near,gave_up,aborted", [
    ("same", 1, 0, 0), ("late", 1, 0, 0), ("other", 0, 0, 0),
    ("nothing", 0, 1, 1), ("aborted", 0, 1, 1),           # the limit, the abort word
    ("none", 0, 0, 0), ("many", 0, 0, 0),                 # not asked; more slices than lanes
])
def test_one_xcd(xcds, what, near, gave_up, aborted):
    result = xcds(what)
    assert result != "unbounded"
    assert [int(x) for x in result.split()[:3]] == [near, gave_up, aborted]


@pytest.mark.parametrize("what,near,gave_up,aborted", [
    ("same", 1, 0, 0), ("late", 1, 0, 0),
    ("other", 0, 0, 0),                                  # one of three slices elsewhere: an answer for all lanes
    ("nothing", 0, 1, 1), ("aborted", 0, 1, 1),
])
def test_one_xcd_of_several_lanes(xcds, what, near, gave_up, aborted):
    # four lanes, three of them with a slice's word
    assert [int(x) for x in xcds(what, "4").split()[:3]] == [near, gave_up, aborted]
