"""Chebyshev moments with room for two blocks of columns but not for the fused kernels' three (MI355X)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2011_02107_amd import binding as B  # noqa: E402
from paper_2011_02107_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu

EPS = 2.220446049250313e-16
DEV = "cuda:0"
MIB = 1 << 20


@pytest.mark.parametrize("nvec", [8, 5])
def test_two_blocks(nvec):
    """The same sums of the same recurrence in another order: up to 2^22 x 8 squares a launch in 256 x 256 partial
    sums, each of 2^9 terms, and the sums of those; orders doubled once.  At 2^22 rows a block of eight columns is
    256 MiB, and 2.5 blocks are left."""
    ctx = B.Context(0)
    L, M = 22, 9
    ham = B.dacp_build_hamiltonian(ctx, L, inputs.ising_chain(L))
    e = ham.info()["sum_abs"]
    g = torch.Generator(device=DEV)
    g.manual_seed(7)
    R = torch.randn(1 << L, nvec, generator=g, device=DEV, dtype=torch.float64)
    want = B.dacp_dos_moments(ctx, ham, e, M, nvec=nvec, R=R)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    left = 80 * nvec  # 2.5 blocks of nvec columns
    filler = []  # the free size read first can fall short of what the device gives
    try:
        for _ in range(8):
            more = torch.cuda.mem_get_info()[0] - left * MIB
            if more < 4 * MIB:
                break
            filler.append(torch.empty(more, dtype=torch.uint8, device=DEV))
        assert torch.cuda.mem_get_info()[0] <= (left + 4) * MIB
        got = B.dacp_dos_moments(ctx, ham, e, M, nvec=nvec, R=R)
    finally:
        del filler
        torch.cuda.empty_cache()
        ham.close()
        ctx.close()
    assert np.abs(got - want).max() <= 2 * (1 << 9) * EPS
