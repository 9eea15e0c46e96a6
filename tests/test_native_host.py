"""Host code that needs the runtime's headers but no device, in harnesses of tests/native/ (CPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2011_02107_amd", "csrc")
NATIVE = os.path.join(ROOT, "tests", "native")
CXX = shutil.which(os.environ.get("CXX", "g++"))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

pytestmark = pytest.mark.skipif(
    CXX is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")),
    reason="no host C++ compiler or HIP headers")


def run(tmp_path, name, *args):
    exe = str(tmp_path / name)
    subprocess.run([CXX, "-std=c++17", "-O1", "-I", CSRC, *args, "-o", exe, "-lpthread"], check=True,
                   capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "0 failures" in r.stdout, r.stderr


def test_worker_contexts_describe_the_callers_device(tmp_path):
    run(tmp_path, "worker_context", "-D__HIP_PLATFORM_AMD__", "-isystem", os.path.join(ROCM, "include"),
        os.path.join(NATIVE, "worker_context_harness.cpp"))


def test_onchip_route_is_the_faster_one(tmp_path):
    run(tmp_path, "onchip_route", os.path.join(NATIVE, "onchip_route_harness.cpp"), os.path.join(CSRC, "host_rules.cpp"))


def test_column_groups_pad_only_where_it_pays(tmp_path):
    run(tmp_path, "column_plan", os.path.join(NATIVE, "column_plan_harness.cpp"), os.path.join(CSRC, "host_rules.cpp"))


def test_secular_roots_against_long_double(tmp_path):
    run(tmp_path, "secular", os.path.join(NATIVE, "secular_harness.cpp"))
