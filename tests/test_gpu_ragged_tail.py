"""Recurrences whose last columns run in a launch of their own, narrower than the others' groups (MI355X).

Columns are independent: a call's are those of the whole groups alone and of the left-over columns alone, which
run the same or the general kernels.  A recurrence of n steps of an operator of norm at most 1 adds rounding
of a few n eps per element of a unit column, in any order of its sums.
"""
import math

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


def unit(L, b):
    g = torch.Generator(device=DEV)
    g.manual_seed(100 * L + b)
    x = torch.randn(1 << L, b, generator=g, device=DEV, dtype=torch.float64)
    return (x / x.norm(dim=0)).contiguous()


@pytest.mark.parametrize("L,b", [(19, 9), (19, 11), (18, 10), (20, 17)])
def test_basis_and_projection(ctx, L, b):
    ham = B.dacp_build_hamiltonian(ctx, L, inputs.ising_chain(L))
    e = ham.info()["sum_abs"]
    n, a_r, full = 1, 0.2, b - b % 8
    x = unit(L, b)
    m = 3 * b

    def basis(cols):
        V = torch.full((1 << L, 3 * cols.shape[1] + 1), 7.0, device=DEV, dtype=torch.float64)
        assert B.dacp_basis(ctx, ham, cols.contiguous(), V, e, a_r * e, n) == 3 * cols.shape[1]
        assert bool((V[:, -1] == 7.0).all())
        return V[:, :-1].reshape(1 << L, 3, -1)

    want = torch.cat([basis(x[:, :full]), basis(x[:, full:])], dim=2)
    steps = math.pi / a_r
    assert (basis(x) - want).abs().max().item() <= 8 * steps * EPS

    V = torch.empty(1 << L, m, device=DEV, dtype=torch.float64)
    S, P = (torch.empty(m, m, device=DEV, dtype=torch.float64) for _ in range(2))
    S1, P1 = torch.empty_like(S), torch.empty_like(P)
    B.dacp_basis_stored_moments(ctx, ham, x, V, S, P, e, a_r * e, n)
    B.dacp_basis_moments(ctx, ham, x, S1, P1, e, a_r * e, n)
    s = V.T.contiguous() @ V
    # sums of 2^L products of unit columns, and moments of up to 2 n + 1 recorded orders
    tol = (2 << L) * EPS + 20 * steps * EPS
    assert (S - s).abs().max().item() <= tol and (S1 - s).abs().max().item() <= tol
    assert (P - P1).abs().max().item() <= 2 * tol * e
    ham.close()


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("L,b", [(19, 9), (19, 12), (20, 10)])
def test_filter(ctx, L, b, precision):
    ham = B.dacp_build_hamiltonian(ctx, L, inputs.ising_chain(L))
    e = ham.info()["sum_abs"]
    a_r, K, full = 0.2, 30, b - b % 8
    x = unit(L, b)

    def run(cols):
        cols = cols.contiguous()
        y = torch.empty_like(cols)
        if precision == "f64":
            B.dacp_filter(ctx, ham, y, e, a_r * e, K, start=cols)
        else:
            B.dacp_filter(ctx, ham, y, e, a_r * e, K, start=cols, precision=B.DACP_F32, fp64_tail=10)
        return y

    want = torch.cat([run(x[:, :full]), run(x[:, full:])], dim=1)
    assert (run(x) - want).abs().max().item() <= 40 * K * (EPS if precision == "f64" else 2.0 ** -24)
    ham.close()


def test_density_moments(ctx):
    L, nvec, M = 19, 11, 9
    ham = B.dacp_build_hamiltonian(ctx, L, inputs.ising_chain(L))
    e = ham.info()["sum_abs"]
    R = unit(L, nvec)
    parts = [R[:, :8].contiguous(), R[:, 8:].contiguous()]
    want = sum(r.shape[1] * B.dacp_dos_moments(ctx, ham, e, M, nvec=r.shape[1], R=r) for r in parts) / nvec
    # squares of 2^19 x 8 elements in 2^16 partial sums, doubled
    assert np.abs(B.dacp_dos_moments(ctx, ham, e, M, nvec=nvec, R=R) - want).max() <= 4 * 64 * EPS + 16 * M * EPS
    ham.close()
