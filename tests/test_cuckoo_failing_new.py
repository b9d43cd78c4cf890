"""The blocked cuckoo table under failing allocations (CPU): an insertion that
is refused with PIR_ENOMEM leaves every message's bytes in its own slot."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_refused_insertions_leave_the_table_whole(tmp_path):
    exe = str(tmp_path / "cuckoo_failing_new")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "include"), "-I/opt/rocm/include",
                    "-D__HIP_PLATFORM_AMD__", "-o", exe, os.path.join(ROOT, "tests", "cuckoo_failing_new.cpp"),
                    os.path.join(ROOT, "paper_2001_08250_amd", "csrc", "cuckoo.cpp")], check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr
