"""Recurrences over several column groups in one launch, with zero columns filling a ragged width.

The filter and the evolution of b columns must equal the general kernels' (knob "fused" = 0) to the
rounding of a few hundred steps, for widths around the group widths and the groups of one launch;
columns of V outside the basis must not be written.  Every stored column has norm at most 1 and a
Chebyshev recurrence of n steps adds rounding of about n eps per element of that size.
"""
import math

import pytest

torch = pytest.importorskip("torch")

from paper_2011_02107_amd import binding as B  # noqa: E402
from paper_2011_02107_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu

EPS = 2.220446049250313e-16


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def unit(L, b):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(100 * L + b)
    x = torch.randn(1 << L, b, generator=g, device="cuda:0", dtype=torch.float64)
    return (x / x.norm(dim=0)).contiguous()


def both(ctx, f):
    out = []
    for fused in (1, 0):
        ctx.tune("fused", fused)
        try:
            out.append(f())
        finally:
            ctx.tune("fused", 1)
    return out


@pytest.mark.parametrize("L,b,group", [(15, 2, 0), (15, 3, 0), (15, 8, 0), (15, 9, 0), (15, 23, 0), (15, 7, 3), (16, 33, 4),
                                       (17, 65, 0), (18, 40, 0)])
def test_basis_groups(ctx, L, b, group):
    ham = B.dacp_build_hamiltonian(ctx, L, inputs.spin_glass(L, 3) if b % 2 else inputs.ising_chain(L))
    e = ham.info()["sum_abs"]
    n, a_r = 2, 0.05
    x = unit(L, b)
    m = b * (2 * n + 1)

    def run():
        V = torch.full((1 << L, m + 3), 7.0, device="cuda:0", dtype=torch.float64)
        assert B.dacp_basis(ctx, ham, x, V, e, a_r * e, n, group=group) == m
        return V

    v1, v0 = both(ctx, run)
    assert bool((v1[:, m:] == 7.0).all())
    assert (v1[:, :m] - v0[:, :m]).abs().max().item() <= 4 * (n * math.pi / a_r) * EPS
    ham.close()


@pytest.mark.parametrize("b", [3, 9, 33])
@pytest.mark.parametrize("moments", ["basis_moments", "stored"])
def test_moment_groups(ctx, b, moments):
    L, n, a_r = 15, 2, 0.05
    ham = B.dacp_build_hamiltonian(ctx, L, inputs.ising_chain(L))
    e = ham.info()["sum_abs"]
    x = unit(L, b)
    m = b * (2 * n + 1)

    def run():
        S = torch.zeros(m, m, device="cuda:0", dtype=torch.float64)
        P = torch.zeros_like(S)
        if moments == "stored":
            V = torch.full((1 << L, m + 1), 7.0, device="cuda:0", dtype=torch.float64)
            B.dacp_basis_stored_moments(ctx, ham, x, V, S, P, e, a_r * e, n)
            assert bool((V[:, m] == 7.0).all())
        else:
            B.dacp_basis_moments(ctx, ham, x, S, P, e, a_r * e, n)
        return S, P

    (s1, p1), (s0, p0) = both(ctx, run)
    steps = 2 * n * math.pi / a_r
    assert (s1 - s0).abs().max().item() <= 20 * steps * EPS
    assert (p1 - p0).abs().max().item() <= 20 * steps * EPS * e
    ham.close()


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("b", [3, 9, 20, 65])
def test_filter_groups(ctx, b, precision):
    L, a_r, K = 15, 0.1, 80
    ham = B.dacp_build_hamiltonian(ctx, L, inputs.ising_chain(L))
    e = ham.info()["sum_abs"]
    x = unit(L, b)

    def run():
        y = torch.empty_like(x)
        if precision == "f64":
            B.dacp_filter(ctx, ham, y, e, a_r * e, K, start=x)
        else:
            B.dacp_filter(ctx, ham, y, e, a_r * e, K, start=x, precision=B.DACP_F32, fp64_tail=30)
        return y

    y1, y0 = both(ctx, run)
    # FP32 part: 50 orders of 2^-24 each, amplified by the filter's growth of the window by at most a few
    tol = 40 * K * EPS if precision == "f64" else 40 * K * 2.0 ** -24
    assert (y1 - y0).abs().max().item() <= tol
    ham.close()
