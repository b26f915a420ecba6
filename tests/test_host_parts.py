"""Host parts of the library built alone with g++ and run on the CPU."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1310_6978_amd", "csrc")


def build_and_run(tmp_path, name):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not found")
    out = str(tmp_path / name)
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-g", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I", CSRC,
                           "-I", os.path.join(ROOT, "include"), "-isystem", "/opt/rocm/include",
                           os.path.join(ROOT, "tests", "host", name + ".cpp"), "-lpthread", "-o", out])
    r = subprocess.run([out], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_list_entry(tmp_path):
    build_and_run(tmp_path, "list_entry")


def test_scratch_pool(tmp_path):
    build_and_run(tmp_path, "scratch_pool")
