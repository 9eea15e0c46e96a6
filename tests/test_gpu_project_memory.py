"""Explicit projection with little memory left on the device (MI355X): column chunks of H V are all it needs."""
import math

import pytest

torch = pytest.importorskip("torch")

from paper_2011_02107_amd import binding as B  # noqa: E402
from paper_2011_02107_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu

EPS = 2.220446049250313e-16
DEV = "cuda:0"
MIB = 1 << 20


def test_projection_fits_the_memory_left():
    """512 columns of 2^14 rows are 64 MiB; the split products' scratch is as much again.  Sums of 2^14 products of
    columns of norm near 1, in another order: D eps, times ||H|| in P."""
    ctx = B.Context(0)
    L, m = 14, 4000
    D = 1 << L
    ham = B.dacp_build_hamiltonian(ctx, L, inputs.ising_chain(L))
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    V = torch.randn(D, m, generator=g, device=DEV, dtype=torch.float64) / math.sqrt(D)
    S, P = (torch.empty(m, m, device=DEV, dtype=torch.float64) for _ in range(2))
    B.dacp_project(ctx, ham, V, S, P)
    want = S.clone(), P.clone()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    filler, left = [], 110
    try:
        for _ in range(8):
            more = torch.cuda.mem_get_info()[0] - left * MIB
            if more < 4 * MIB:
                break
            filler.append(torch.empty(more, dtype=torch.uint8, device=DEV))
        assert torch.cuda.mem_get_info()[0] <= (left + 4) * MIB
        B.dacp_project(ctx, ham, V, S, P)
        torch.cuda.synchronize()
    finally:
        del filler
        torch.cuda.empty_cache()
    e = ham.info()["sum_abs"]
    assert (S - want[0]).abs().max().item() <= 2 * D * EPS
    assert (P - want[1]).abs().max().item() <= 2 * D * EPS * e
    ham.close()
    ctx.close()
