"""On-chip column kernels for Hamiltonians without single-spin flips: the paper's X_i X_j models, and pairs with
signs (MI355X).  Against the recurrences written out in torch FP64: n applies of an operator of norm at most 1 add
rounding of a few n eps per element of a unit column.
"""
import math
import time

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


def terms(kind, L):
    if kind == "xx":
        return inputs.paper_sgs(L, 7)
    rng = np.random.default_rng(L)
    ops = [(inputs.X, inputs.X), (inputs.Y, inputs.Y), (inputs.X, inputs.Z), (inputs.Z, inputs.X)]
    return inputs.make_terms([ops[(i + j) % 4][0:1] + (i,) + ops[(i + j) % 4][1:2] + (j, rng.uniform(-1, 1))
                              for i in range(L) for j in range(i + 1, L)])


def plain(t, L):
    s = torch.arange(1 << L, device=DEV)

    def parity(v):
        p = torch.zeros_like(v)
        for _ in range(15):
            p ^= v & 1
            v = v >> 1
        return 1.0 - 2.0 * p.double()

    def apply(v):
        y = torch.zeros_like(v)
        for r in t:
            x = z = ny = 0
            for op, site in ((int(r["op_a"]), int(r["site_a"])), (int(r["op_b"]), int(r["site_b"]))):
                x ^= (1 << site) if op in (inputs.X, inputs.Y) else 0
                z ^= (1 << site) if op in (inputs.Z, inputs.Y) else 0
                ny += op == inputs.Y
            c = float(r["coeff"]) * (-1.0 if ny == 2 else 1.0)
            y += c * parity((s ^ x) & z)[:, None] * v[s ^ x]
        return y

    return apply


def unit(D, b):
    g = torch.Generator(device=DEV)
    g.manual_seed(D + b)
    x = torch.randn(D, b, generator=g, device=DEV, dtype=torch.float64)
    return (x / x.norm(dim=0)).contiguous()


@pytest.mark.parametrize("kind", ["xx", "signed"])
@pytest.mark.parametrize("L", [2, 5, 9, 10, 11, 12, 13, 14])
def test_basis_filter_and_moments(ctx, L, kind):
    t = terms(kind, L)
    ham = B.dacp_build_hamiltonian(ctx, L, t)
    h = plain(t, L)
    D, n, a_r = 1 << L, 2, 0.3
    b = 300 if L >= 13 else 3  # enough columns for the on-chip route at every size
    e = 1.05 * ham.info()["sum_abs"]
    x = unit(D, b)
    m = b * (2 * n + 1)
    V = torch.empty(D, m, device=DEV, dtype=torch.float64)
    assert B.dacp_basis(ctx, ham, x, V, e, a_r * e, n) == m
    ks = [2 * math.floor(j * math.pi / (2 * a_r)) for j in range(1, n + 1)]
    ref = [x, h(x) / e]
    while len(ref) <= ks[-1]:
        ref.append(h(ref[-1]) * (2.0 / e) - ref[-2])
    want = torch.cat([x] + [ref[k + d] for k in ks for d in (-1, 0)], dim=1)
    assert (V - want).abs().max().item() <= 8 * ks[-1] * EPS

    a, K = a_r * e, 12
    ec, e0 = 0.5 * (e * e + a * a), 0.5 * (e * e - a * a)
    rho = math.exp(math.acosh(1 + 2 * a * a / (e * e - a * a)))
    t0, t1 = x, (h(h(x)) - ec * x) / (e0 * rho)
    for _ in range(1, K):
        t0, t1 = t1, (h(h(t1)) - ec * t1) * (2 / (e0 * rho)) - t0 / rho ** 2
    want = t1 / t1.norm(dim=0)
    lost = 1.0 / t1.norm(dim=0).min().item()  # the filter's damping of the start's norm
    for precision, tail, eps in ((B.DACP_F64, 0, EPS), (B.DACP_F32, 5, 2.0 ** -24)):
        y = torch.empty_like(x)
        B.dacp_filter(ctx, ham, y, e, a, K, start=x, precision=precision, fp64_tail=tail)
        assert (y - want).abs().max().item() <= 16 * K * eps * max(1.0, lost)

    M = 7
    mu = B.dacp_dos_moments(ctx, ham, e, M, nvec=b, R=x)
    want = [float((x * ref[k]).sum()) / b for k in range(M)]
    assert np.abs(mu - np.array(want)).max() <= 16 * M * EPS
    ham.close()


def test_time_of_a_pair_flip(ctx):
    """A column's apply at 2^14 rows took 11 (sgs) and 2.4 (tfim) times the chain's while each flip's table entry
    was waited for and single-spin sweeps ran with coefficients of zero; 7.5 and 1.5 times without.  256 columns
    are one per compute unit."""
    L, b, K = 14, 256, 200
    x, y = unit(1 << L, b), torch.empty(1 << L, b, device=DEV, dtype=torch.float64)

    def seconds(t):
        ham = B.dacp_build_hamiltonian(ctx, L, t)
        e = ham.info()["sum_abs"]
        best = math.inf
        for _ in range(4):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            B.dacp_filter(ctx, ham, y, e, 0.1 * e, K, start=x)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        ham.close()
        return best

    chain = seconds(inputs.ising_chain(L))
    assert seconds(inputs.paper_sgs(L, 3)) <= 9.2 * chain
    assert seconds(inputs.paper_tfim(L, 3)) <= 1.9 * chain
