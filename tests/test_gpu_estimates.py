"""Spectral estimates whose scalars stay on the device: Chebyshev moments past the on-chip route's reach (MI355X)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2011_02107_amd import binding as B  # noqa: E402
from paper_2011_02107_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu

EPS = 2.220446049250313e-16
DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def test_moments_of_a_start_block_past_4_gib(ctx):
    """Moments are averages over the vectors' <r, T_k r>, so a block's are its halves' weighted by <r, r>.
    The halves' offsets fit 32 bits, the block's do not.  The sums are of 2^14 x 40000 squares in at most
    2^16 partial sums of 10000 terms, each rounding to n eps; twice that for the factor 2 of the doubled orders."""
    L, nvec, M = 14, 40000, 6
    ham = B.dacp_build_hamiltonian(ctx, L, inputs.ising_chain(L))
    e = ham.info()["sum_abs"]
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    R = torch.randn(1 << L, nvec, generator=g, device=DEV, dtype=torch.float64)
    mu = B.dacp_dos_moments(ctx, ham, e, M, nvec=nvec, R=R)
    want, total = np.zeros(M), 0.0
    for half in (R[:, : nvec // 2].contiguous(), R[:, nvec // 2:].contiguous()):
        n0 = float((half * half).sum())
        want += n0 * B.dacp_dos_moments(ctx, ham, e, M, nvec=half.shape[1], R=half)
        total += n0
    assert np.abs(mu - want / total).max() <= 2 * 10000 * EPS
    ham.close()
