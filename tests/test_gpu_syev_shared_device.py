"""Dense eigensolvers in two processes on one device (MI355X): the runtime gives cooperative launches to one of them
at a time, and the other solves in memory."""
import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")

from paper_2011_02107_amd import binding as B  # noqa: E402

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOLVE = """
import numpy as np, torch
from paper_2011_02107_amd import binding as B, inputs
EPS = 2.220446049250313e-16
ctx = B.Context(0)
def symmetric(n):
    a = np.random.default_rng(n).standard_normal((n, n))
    return a + a.T
def check(a, w, z):
    # 20 n eps ||A||, as for the register form
    n, ref = len(w), np.linalg.eigvalsh(a)
    norm = np.abs(ref).max()
    assert np.abs(w - ref).max() <= 20 * n * EPS * norm, n
    if z is not None:
        v = z.cpu().numpy()
        assert np.abs(v @ a - w[:, None] * v).max() <= 20 * n * EPS * norm, n
        assert np.abs(v @ v.T - np.eye(n)).max() <= 20 * n * EPS, n
def single(n, vectors):
    a = symmetric(n)
    d = torch.as_tensor(a, device="cuda:0")
    z = torch.empty_like(d) if vectors else None
    check(a, B.dacp_syev(ctx, d, z), z)
def batch(sizes):
    a = [symmetric(n) for n in sizes]
    d = [torch.as_tensor(x, device="cuda:0") for x in a]
    z = [torch.empty_like(x) for x in d]
    for x, w, y in zip(a, B.dacp_syev_batched(ctx, d, z), z):
        check(x, w, y)
for n, vectors in ((40, True), (300, True), (300, False), (1100, True)):
    single(n, vectors)
batch((3, 64, 200, 350))
batch((700, 2))
batch([150 + i for i in range(12)])
for L in (9, 10):
    ham = B.dacp_build_hamiltonian(ctx, L, inputs.spin_glass(L, 4))
    got = B.dacp_central_eigs_batched(ctx, [ham], 20, B.default_opts(b=8, seed=2))[0][0]
    alone = B.dacp_central_eigs(ctx, ham, 20, B.default_opts(b=8, seed=2))[0]
    assert np.abs(np.asarray(got) - np.asarray(alone)).max() <= 2e-10 * ham.info()["sum_abs"]
print("solved", flush=True)
"""


def test_second_process():
    """The first has launched cooperatively and stays; neither it nor the second one fails."""
    ctx = B.Context(0)
    a = torch.eye(300, device="cuda:0", dtype=torch.float64)
    assert B.dacp_syev(ctx, a, None)[0] == 1.0
    r = subprocess.run([sys.executable, "-c", SOLVE], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip() == "solved", r.stderr[-2000:]
    a = torch.eye(300, device="cuda:0", dtype=torch.float64)
    assert B.dacp_syev(ctx, a, None)[0] == 1.0
    ctx.close()
