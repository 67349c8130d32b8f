"""The reading of tables into host memory (csrc/host_copy.h) on the CPU, against a stub of the runtime whose copies happen later
on another thread: sizes at the edges of blocks, fewer threads and none, no pinned memory, destinations that are not pageable
memory, and an error at any call."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2505_09258_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_host_copy_against_a_stub_runtime(tmp_path):
    exe = tmp_path / "host_copy_check"
    native = os.path.join(HERE, "native")
    subprocess.run(["g++", "-std=c++17", "-O2", "-pthread", "-I", native, "-I", CSRC, os.path.join(native, "host_copy_check.cpp"),
                    "-o", str(exe), "-ldl"], check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
