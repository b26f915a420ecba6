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


def test_registers_in_lds_are_aligned(tmp_path):
    """The jump-table form moves a lane's 16 words between its LDS registers and
    the VGPRs 16 bytes at a time: whatever a kernel keeps in LDS in front of
    them, they start at a multiple of 16."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    src = tmp_path / "kernels.hip"
    src.write_text('#include "fbg_device.h"\n'
                   "template __global__ void fbg::dev::k_batch<4, 3, fbg::dev::MODE_COUNT>(fbg::BatchArgs);\n"
                   "template __global__ void fbg::dev::k_batch<4, 1, fbg::dev::MODE_COUNT>(fbg::BatchArgs);\n"
                   "template __global__ void fbg::dev::k_eval<4, fbg::dev::MODE_ENUM, 1>(fbg::EvalArgs);\n")
    out = tmp_path / "kernels.s"
    subprocess.check_call([hipcc, "-x", "hip", "--offload-arch=gfx950", "--offload-device-only", "-S", "-O1",
                           "-std=c++17", "-w", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-mllvm",
                           "-structurizecfg-skip-uniform-regions=true", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                           str(src), "-o", str(out)])
    sizes = [int(line.split()[-1]) for line in out.read_text().splitlines() if ".amdhsa_group_segment_fixed_size" in line]
    assert len(sizes) == 3 and all(s % 16 == 0 for s in sizes), sizes
