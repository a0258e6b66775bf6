"""Host plans of the kernels, checked by small C++ programs built from the library's
sources with g++ (no GPU code involved)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1612_08091_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

pytestmark = [
    pytest.mark.skipif(shutil.which("g++") is None, reason="no g++"),
    pytest.mark.skipif(not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime_api.h")),
                       reason="HIP headers not found"),
]


def run_check(tmp_path, name, *sources):
    exe = str(tmp_path / name)
    cmd = ["g++", "-std=c++17", "-O2", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I" + CSRC,
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROCM, "include"),
           os.path.join(ROOT, "tests", "host", name + ".cpp")]
    cmd += [os.path.join(CSRC, s) for s in sources] + ["-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout[-2000:] + r.stderr[-2000:]
    return r.stdout


def test_xcd_split(tmp_path):
    run_check(tmp_path, "xcd_split_check")


def test_pauli_plan(tmp_path):
    run_check(tmp_path, "pauli_plan_check", "pauli_plan.cpp")


def test_plan_weights(tmp_path):
    run_check(tmp_path, "plan_weights_check", "planner.cpp")


def test_table_groups(tmp_path):
    run_check(tmp_path, "table_groups_check", "planner.cpp", "tileprog.cpp")
