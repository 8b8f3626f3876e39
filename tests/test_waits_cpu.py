"""The wait loops of the persistent kernels as host code: every wait ends, whatever is or is not written."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def waits(tmp_path_factory):
    clang = shutil.which("amdclang++") or "/opt/rocm/llvm/bin/clang++"   # (the sources use vector extensions that g++ lacks)
    if not os.path.exists(clang):
        pytest.skip("no clang++")
    out = str(tmp_path_factory.mktemp("waits") / "waits")
    subprocess.run([clang, "-x", "c++", "-std=c++17", "-O1", "-Wno-everything", "-I", os.path.join(HERE, "wave_on_cpu"), "-I", os.path.join(os.path.dirname(HERE), "paper_1904_04956_amd", "csrc"),
                    os.path.join(HERE, "wave_on_cpu", "waits.cpp"), "-o", out], check=True)
    return lambda *what: subprocess.run([out, *what], capture_output=True, text=True, timeout=60, check=True).stdout.strip()


@pytest.mark.parametrize("what,gave_up,aborted", [
    ("there", 0, 0), ("late", 0, 0), ("given up", 1, 0),
    ("nothing", 1, 1),                                   # the limit
    ("rest", 1, 1),                                      # the limit with one element missing
    ("rest, aborted", 1, 1),                             # the abort word
])
def test_every_wait_for_a_tile_ends(waits, what, gave_up, aborted):
    result = waits(what)
    assert result != "unbounded"
    r, word, loads, whole = (int(x) for x in result.split())
    assert (r, word) == (gave_up, aborted) and whole == (not gave_up)
    assert (loads == 0) == (what in ("there", "given up"))


@pytest.mark.parametrize("what,gave_up,aborted", [
    ("there", 0, 0), ("late", 0, 0), ("given up", 1, 0),
    ("nothing", 1, 1),                                   # the limit
    ("rest", 1, 1),                                      # the limit with one element missing
    ("rest, aborted", 1, 1),                             # the abort word
])
def test_every_wait_of_the_kernels_for_few_sequences_ends(waits, what, gave_up, aborted):
    result = waits(what, "few")
    assert result != "unbounded"
    r, word, loads, whole = (int(x) for x in result.split())
    assert (r, word) == (gave_up, aborted) and whole == (not gave_up)


@pytest.mark.parametrize("what,gave_up,aborted", [
    ("there", 0, 0), ("late", 0, 0), ("given up", 1, 0),
    ("nothing", 1, 1),                                   # the limit
    ("rest", 1, 1),                                      # the limit with one word missing
    ("rest, aborted", 1, 1),                             # the abort word
])
def test_every_wait_of_the_float_kernels_ends(waits, what, gave_up, aborted):
    result = waits(what, "float")
    assert result != "unbounded"
    r, word, loads, whole = (int(x) for x in result.split())
    assert (r, word) == (gave_up, aborted) and whole == (not gave_up)
    assert (loads == 0) == (what in ("there", "given up"))
