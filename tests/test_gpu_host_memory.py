"""A failed host allocation inside the dense eigensolvers ends in a status at the C entry (MI355X).

In a child process that preloads a failing operator new: the divide and conquer's tables of a matrix of
2900 rows and more are above 200 KB, and so is the job list of 8192 matrices.
"""
import os
import shutil
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = shutil.which(os.environ.get("CXX", "g++"))

CHILD = """
import ctypes, sys
import numpy as np, torch
from paper_2011_02107_amd import binding as B
fail = ctypes.CDLL(None).fail_new_at
fail.argtypes = [ctypes.c_size_t]
ctx = B.Context(0)
def failing(call):
    fail(200000)
    try:
        call()
        return 0
    except B.DacpError as e:
        return e.status
    finally:
        fail(0)
for n in (2900, 3100):
    lam = np.linspace(-1.0, 1.0, n)
    a = torch.diag(torch.as_tensor(lam, device="cuda:0"))
    work, z = a.clone(), torch.empty_like(a)
    print(n, failing(lambda: B.dacp_syev(ctx, work, z)), flush=True)
    work.copy_(a)
    print(n, np.abs(B.dacp_syev(ctx, work, z) - lam).max() < 1e-12, flush=True)
one = [torch.ones(1, 1, dtype=torch.float64, device="cuda:0")] * 8192
print("list", failing(lambda: B.dacp_syev_batched(ctx, one, one)), flush=True)
"""


@pytest.mark.skipif(CXX is None, reason="no host C++ compiler")
def test_failed_host_allocation_is_a_status(tmp_path):
    so = str(tmp_path / "fail_new.so")
    subprocess.run([CXX, "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "native", "fail_new.cpp"),
                    "-o", so], check=True, capture_output=True, text=True)
    preload = ":".join(p for p in (os.environ.get("LD_PRELOAD", ""), so) if p)
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, env=dict(os.environ, LD_PRELOAD=preload),
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.split("\n")[:5] == ["2900 -2", "2900 True", "3100 -2", "3100 True", "list -2"]
