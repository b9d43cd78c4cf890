"""The library's host code over a HIP runtime in host memory (CPU only): what it
allocates, copies, captures and launches. Kernels do not run here."""
import os
import shutil
import subprocess

import pytest

import paper_2001_08250_amd as pir

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def fake_hip(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("fake_hip") / "fake_hip")
    lib = os.path.dirname(pir.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + os.path.dirname(pir.HEADER), "-I/opt/rocm/include",
                    "-D__HIP_PLATFORM_AMD__", "-o", exe, os.path.join(HERE, "fake_hip.cpp"), "-L" + lib,
                    "-l:" + os.path.basename(pir.LIB_PATH), "-Wl,-rpath," + lib, "-rdynamic", "-Wl,--allow-shlib-undefined"],
                   check=True)
    return exe


@pytest.mark.parametrize("scenario", ["first_read", "read_without_pinned_memory", "code_without_pinned_memory",
                                      "tuned_leaves", "stream_plans", "answer_scratch"])
def test_host_paths(fake_hip, scenario):
    run = subprocess.run([fake_hip, scenario], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr
