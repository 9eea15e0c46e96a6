"""Dense eigensolvers when the register tridiagonalisation's exchange times out (MI355X): every workgroup's wait is
bounded, here by no poll at all, and the matrices go column by column."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2011_02107_amd import binding as B  # noqa: E402
from paper_2011_02107_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu

EPS = 2.220446049250313e-16
DEV = "cuda:0"


@pytest.fixture()
def ctx():
    c = B.Context(0)
    c.tune("tri_spins", 0)
    yield c
    torch.cuda.synchronize()
    c.close()


def symmetric(n):
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    a = torch.randn(n, n, generator=g, device=DEV, dtype=torch.float64)
    return (a + a.T).contiguous()


def check(a, w, z):
    """20 n eps ||A||, as for the register form."""
    n = a.shape[0]
    w = torch.as_tensor(w, device=DEV)
    norm = w.abs().max().item()
    assert (torch.linalg.eigvalsh(a.cpu()).to(DEV) - w).abs().max().item() <= 20 * n * EPS * norm
    if z is not None:
        assert (z @ a - w[:, None] * z).abs().max().item() <= 20 * n * EPS * norm
        assert (z @ z.T - torch.eye(n, device=DEV, dtype=torch.float64)).abs().max().item() <= 20 * n * EPS


@pytest.mark.parametrize("n,vectors", [(5, True), (40, True), (300, True), (300, False), (1100, True)])
def test_syev(ctx, n, vectors):
    a = symmetric(n)
    z = torch.empty_like(a) if vectors else None
    check(a, B.dacp_syev(ctx, a.clone(), z), z)


def test_syev_batched(ctx):
    a = [symmetric(n) for n in (3, 64, 200, 350)]
    z = [torch.empty_like(x) for x in a]
    for x, w, y in zip(a, B.dacp_syev_batched(ctx, [x.clone() for x in a], z), z):
        check(x, w, y)


def test_batched_realisations(ctx):
    """Through the workers' contexts and the shared solver's stream."""
    hams = [B.dacp_build_hamiltonian(ctx, 10, inputs.spin_glass(10, 40 + i)) for i in range(3)]
    o = B.default_opts(b=8, seed=2)
    got = B.dacp_central_eigs_batched(ctx, hams, 30, o)[0]
    ctx.tune("tri_spins", 1 << 24)
    want = B.dacp_central_eigs_batched(ctx, hams, 30, o)[0]
    for g, w, h in zip(got, want, hams):
        assert np.abs(np.asarray(g) - np.asarray(w)).max() <= 2e-10 * h.info()["sum_abs"]
        h.close()
