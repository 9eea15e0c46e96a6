"""dacp_autotune times the kernels whose knobs it sets, not the on-chip route (MI355X)."""
import math
import time

import pytest

torch = pytest.importorskip("torch")

from paper_2011_02107_amd import binding as B  # noqa: E402
from paper_2011_02107_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu


def test_autotune_times_the_memory_recurrence():
    """At 8 spins a step takes a launch or two, at least 3 us; on chip it takes 1 (dacp_basis does).  Timed
    there, every knob setting was the same kernel and the first one of the widest group won."""
    ctx = B.Context(0)
    L, b = 8, 1
    ham = B.dacp_build_hamiltonian(ctx, L, inputs.ising_chain(L))
    _, tuned = B.dacp_autotune(ctx, ham, b=b, steps=400)
    e = ham.info()["sum_abs"]
    steps, n = 4000, 1
    x = torch.randn(1 << L, b, device="cuda:0", dtype=torch.float64)
    V = torch.empty(1 << L, 3 * b, device="cuda:0", dtype=torch.float64)
    best = math.inf
    for _ in range(5):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        B.dacp_basis(ctx, ham, x, V, e, e * math.pi / steps, n)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) * 1e6 / steps)
    assert tuned > 1.5 * best
    ham.close()
    ctx.close()
