"""The fenced protocol's releases in the built kernels: the write-back of the L2 is waited for before the counter that says so.  The
compiler writes that wait only while it counts something in flight; a store written in assembly it does not count."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_1904_04956_amd import binding

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"


def test_every_release_waits_for_its_write_back(tmp_path):
    if not (os.path.exists(OBJDUMP) and os.path.exists(binding.LIB_PATH)):
        pytest.skip("no llvm-objdump, or nothing built")
    lib = shutil.copy(binding.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    releases, missing = {}, []
    for code in glob.glob(str(tmp_path / "*gfx950")):
        if os.path.getsize(code) == 0:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", code], check=True, capture_output=True, text=True).stdout
        name, waiting = "", False
        for line in text.splitlines():
            head = re.match(r"[0-9a-f]+ <(.*)>:$", line)
            if head:
                name, waiting = head[1], False
                continue
            op = line.split("//")[0].strip()
            if op.startswith("buffer_wbl2"):
                releases[name] = releases.get(name, 0) + 1
                waiting = True
            elif waiting and op.startswith("s_waitcnt") and "vmcnt(0)" in op:
                waiting = False
            elif waiting and "atomic_add" in op:
                missing.append(name)
                waiting = False
    assert not missing, sorted(set(missing))
    for family in ("rec_fwd_kernelILi256ELb0", "rec_bwd_kernelILi256ELb0", "tile_rec_fwd_kernelILi4ELi16ELb0", "tile_rec_bwd_kernelILi4ELi16ELb0", "multi_tile_rec_bwd_kernelILi4ELi16ELb0"):
        assert any(family in n for n in releases), family
