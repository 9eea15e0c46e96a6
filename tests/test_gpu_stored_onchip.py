"""Stored moments up to 14 spins on both routes (MI355X): basis, S and P on chip (few flips) and through memory (the
spin glass of pair flips with few columns), against the evolution and the products in torch FP64."""
import math

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


@pytest.mark.parametrize("L,model,b", [(5, "chain", 1), (9, "glass", 3), (11, "chain", 6), (13, "tfim", 2), (14, "glass", 4),
                                       (14, "sgs", 2), (14, "tfim", 1)])
def test_stored_moments(ctx, L, model, b):
    t = inputs.ising_chain(L) if model == "chain" else {"glass": inputs.spin_glass, "tfim": inputs.paper_tfim,
                                                        "sgs": inputs.paper_sgs}[model](L, 4)
    ham = B.dacp_build_hamiltonian(ctx, L, t)
    e = ham.info()["sum_abs"]
    D, n, a_r = 1 << L, 2, 0.25
    g = torch.Generator(device=DEV)
    g.manual_seed(L)
    x = torch.randn(D, b, generator=g, device=DEV, dtype=torch.float64)
    x = (x / x.norm(dim=0)).contiguous()
    m = b * (2 * n + 1)
    V = torch.full((D, m + 1), 7.0, device=DEV, dtype=torch.float64)
    S, P = (torch.empty(m, m, device=DEV, dtype=torch.float64) for _ in range(2))
    assert B.dacp_basis_stored_moments(ctx, ham, x, V, S, P, e, a_r * e, n) == m

    def h(v):
        y = torch.empty_like(v)
        B.dacp_apply(ctx, ham, v.contiguous(), y)
        return y

    # the uniform grid: panels 0, k - 1, k for k = delta, 2 delta, delta = 2 floor(pi / (2 a_r))
    delta = max(2, 2 * math.floor(math.pi / (2 * a_r)))
    ref = [x, h(x) / e]
    while len(ref) <= n * delta:
        ref.append(h(ref[-1]) * (2.0 / e) - ref[-2])
    want = torch.cat([x] + [ref[j * delta + d] for j in (1, 2) for d in (-1, 0)], dim=1)
    assert bool((V[:, m] == 7.0).all())
    steps = n * delta
    assert (V[:, :m] - want).abs().max().item() <= 8 * steps * EPS
    # sums of D products of unit columns, through moments of up to 2 n recorded orders
    tol = (2 * D + 40 * steps) * EPS
    assert (S - want.T @ want).abs().max().item() <= tol
    assert (P - want.T @ torch.cat([h(want[:, i:i + 1]) for i in range(m)], dim=1)).abs().max().item() <= tol * e
    ham.close()
