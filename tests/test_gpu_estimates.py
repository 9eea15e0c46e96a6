"""Spectral estimates whose scalars stay on the device: Lanczos bound and Chebyshev moments on chip and, from 15
spins on or past the on-chip route's reach, through memory (MI355X)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import hamiltonian, spectral  # noqa: E402
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


MODELS = {"chain": inputs.ising_chain, "glass": lambda L: inputs.spin_glass(L, 5), "pairs": lambda L: inputs.paper_tfim(L, 5),
          "all_pairs": lambda L: inputs.paper_sgs(L, 5)}


@pytest.mark.parametrize("L,model,steps", [(15, "chain", 1), (15, "chain", 37), (15, "pairs", 20), (16, "glass", 60),
                                           (14, "all_pairs", 12), (12, "all_pairs", 12)])
def test_lanczos_bound(ctx, L, model, steps):
    """The extreme Ritz values of the same recurrence; the bound from residuals is only as good as they are
    converged, so it is compared loosely and against the Ritz values."""
    t = MODELS[model](L)
    v0 = np.random.default_rng(L).standard_normal(1 << L) * 3.0
    ham = B.dacp_build_hamiltonian(ctx, L, t)
    e, lo, hi = B.dacp_spectral_bound(ctx, ham, steps, v0=torch.as_tensor(v0, device=DEV))
    al, be = spectral.lanczos(lambda X: hamiltonian.apply_h(L, t, X), v0, steps)
    ref, theta = spectral.lanczos_bound(al, be, hamiltonian.sum_abs_coeff(t))
    scale = np.abs(theta).max()
    assert abs(lo - theta[0]) <= 1e-9 * scale and abs(hi - theta[-1]) <= 1e-9 * scale
    assert abs(e - ref) <= 1e-6 * ref and e >= max(-lo, hi)
    ham.close()


@pytest.mark.parametrize("L", [9, 15])
@pytest.mark.parametrize("invariant", [1, 2])
def test_lanczos_breakdown(ctx, L, invariant):
    """A start vector in an invariant subspace of 1 or 2 basis states of a Hamiltonian with one flip: the residual
    vanishes after as many steps, and what the device computed from its zero is not used."""
    z = [(inputs.Z, i, inputs.I, 0, 1.0 + 0.25 * i) for i in range(1, L)]  # spin 0 has no field
    ham = B.dacp_build_hamiltonian(ctx, L, inputs.make_terms(z + [(inputs.X, 0, inputs.I, 0, 0.5)]))
    v0 = torch.zeros(1 << L, device=DEV, dtype=torch.float64)
    v0[0] = 2.0
    if invariant == 1:
        v0[1] = 2.0  # the eigenvector of sigma^x_0
    e, lo, hi = B.dacp_spectral_bound(ctx, ham, 20, v0=v0)
    c = sum(1.0 + 0.25 * i for i in range(1, L))
    want = (c + 0.5, c + 0.5) if invariant == 1 else (c - 0.5, c + 0.5)
    # powers of two throughout, but for the normalisation by sqrt(8)
    assert abs(lo - want[0]) <= 16 * EPS * c and abs(hi - want[1]) <= 16 * EPS * c
    assert np.isfinite(e) and e >= hi - 16 * EPS * c
    with pytest.raises(B.DacpError) as err:
        B.dacp_spectral_bound(ctx, ham, 20, v0=torch.zeros_like(v0))
    assert err.value.status == -1
    ham.close()


@pytest.mark.parametrize("L,model,nvec,M", [(15, "chain", 3, 33), (15, "chain", 9, 2), (15, "chain", 1, 1), (15, "pairs", 3, 8),
                                            (16, "glass", 11, 17), (18, "chain", 9, 5), (14, "all_pairs", 2, 9),
                                            (13, "all_pairs", 5, 6)])
def test_density_moments(ctx, L, model, nvec, M):
    """Odd and even numbers of moments and widths that fill no group, against the three-term recurrence: rounding of
    a few M eps, and of sums of 2^L nvec squares in partial sums of at most 2^7 terms."""
    t = MODELS[model](L)
    ham = B.dacp_build_hamiltonian(ctx, L, t)
    e = ham.info()["sum_abs"]
    R = np.random.default_rng(L + M).standard_normal((1 << L, nvec))
    mu = B.dacp_dos_moments(ctx, ham, e, M, nvec, R=torch.as_tensor(R, device=DEV))
    ref = spectral.kpm_moments(lambda X: hamiltonian.apply_h(L, t, X), R, e, M)
    assert len(mu) == M and np.abs(mu - ref).max() <= 2 * (128 + 16 * M) * EPS
    ham.close()
