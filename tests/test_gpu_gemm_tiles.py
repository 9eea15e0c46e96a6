"""FP64 GEMM and projection where the tile walk and the K split change (MI355X).

Outputs of one tile, a partial last tile, one and several bands of 8 tile rows, 64 and 128 wide
tiles, and K split over several ranges.  Every operand and coupling is a small whole number, so each
product is exact in FP64 in any summation order and must equal torch's.
"""
import pytest

torch = pytest.importorskip("torch")

from paper_2011_02107_amd import binding as B  # noqa: E402
from paper_2011_02107_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu

@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def whole(*shape):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(sum(shape))
    return torch.randint(-3, 4, shape, generator=g, device="cuda:0").double()


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (63, 65, 17), (64, 128, 16), (200, 1, 33), (129, 1100, 40), (1100, 513, 100),
                                   (2100, 2050, 70)])
def test_gemm_tile_walk(ctx, ta, tb, M, N, K):
    A = whole(K, M) if ta else whole(M, K)
    Bm = whole(N, K) if tb else whole(K, N)
    C = whole(M, N)
    # the transposed operand is laid out anew for the reference
    ref = -0.5 * (A.T.contiguous() if ta else A) @ (Bm.T.contiguous() if tb else Bm) + 2.0 * C
    B.dacp_gemm(ctx, ta, tb, A, Bm, C, alpha=-0.5, beta=2.0)
    assert torch.equal(C, ref)


@pytest.mark.parametrize("splitk", [0, 1])
@pytest.mark.parametrize("m", [1, 65, 128, 129, 700, 1030, 2900])
def test_project_tile_walk(ctx, m, splitk):
    L = 12
    ham = B.dacp_build_hamiltonian(ctx, L, inputs.ising_chain(L, hx=2.0, hz=1.0))
    V = whole(1 << L, m)
    S = torch.full((m, m), float("nan"), device="cuda:0", dtype=torch.float64)
    P = S.clone()
    ctx.tune("project_splitk", splitk)
    try:
        B.dacp_project(ctx, ham, V, S, P)
        HV = torch.empty_like(V)
        B.dacp_apply(ctx, ham, V, HV)
    finally:
        ctx.tune("project_splitk", 1)
    Vt = V.T.contiguous()
    assert torch.equal(S, Vt @ V)
    assert torch.equal(P, Vt @ HV)
    ham.close()
