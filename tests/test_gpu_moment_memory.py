"""Moment-mode projection with little memory left on the device (MI355X).

The mode serves states too long to store a basis: three blocks of a column group, G psi_E and small
tables are all it needs.  At 2^20 rows a column is 8 MiB; eight columns a group make 192 MiB of blocks.
"""
import pytest

torch = pytest.importorskip("torch")

from paper_2011_02107_amd import binding as B  # noqa: E402
from paper_2011_02107_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu

EPS = 2.220446049250313e-16
DEV = "cuda:0"
MIB = 1 << 20


@pytest.fixture(scope="module")
def call():
    ctx = B.Context(0)
    L, b, n, a_r = 20, 8, 1, 0.3
    D, m = 1 << L, b * (2 * n + 1)
    ham = B.dacp_build_hamiltonian(ctx, L, inputs.ising_chain(L))
    e = ham.info()["sum_abs"]
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    x = torch.randn(D, b, generator=g, device=DEV, dtype=torch.float64)
    x = (x / x.norm(dim=0)).contiguous()
    S = torch.empty(m, m, device=DEV, dtype=torch.float64)
    P = torch.empty_like(S)

    def run():
        B.dacp_basis_moments(ctx, ham, x, S, P, e, a_r * e, n)
        return S.clone(), P.clone()

    yield run, D, e
    torch.cuda.synchronize()
    ham.close()
    ctx.close()


@pytest.mark.parametrize("left", [1200, 440, 380, 310],
                         ids=["fewer_staged", "one_group_staged", "not_staged", "factors_apart"])
def test_moments_fit_the_memory_left(call, left):
    """The same moments in another order of summation: products of unit columns over D rows, D eps each,
    two of them in an entry of S, times e_bound in P."""
    run, D, e = call
    want = run()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    filler = []  # the free size read first can fall short of what the device gives
    try:
        for _ in range(8):
            more = torch.cuda.mem_get_info()[0] - left * MIB
            if more < 4 * MIB:
                break
            filler.append(torch.empty(more, dtype=torch.uint8, device=DEV))
        assert torch.cuda.mem_get_info()[0] <= (left + 4) * MIB
        got = run()
    finally:
        del filler
        torch.cuda.empty_cache()
    assert (got[0] - want[0]).abs().max().item() <= 2 * D * EPS
    assert (got[1] - want[1]).abs().max().item() <= 2 * D * EPS * e
