"""Statuses of the dense eigensolvers for matrices that are not finite (MI355X): no convergence where QR iteration
is the documented method, the numeric status where divide and conquer gives the eigenvectors."""
import pytest

torch = pytest.importorskip("torch")

from paper_2011_02107_amd import binding as B  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def status(call):
    with pytest.raises(B.DacpError) as err:
        call()
    return err.value.status


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("n,vectors,want", [(3, True, -7), (40, True, -7), (200, True, -6), (200, False, -7)])
def test_syev(ctx, n, vectors, want, bad):
    a = torch.eye(n, device="cuda:0", dtype=torch.float64)
    a[0, n - 1] = a[n - 1, 0] = bad
    z = torch.empty_like(a) if vectors else None
    assert status(lambda: B.dacp_syev(ctx, a, z)) == want


@pytest.mark.parametrize("noalloc", [False, True])
def test_syev_batched(ctx, noalloc):
    a = [torch.eye(n, device="cuda:0", dtype=torch.float64) for n in (33, 200)]
    a[1][3, 2] = a[1][2, 3] = float("nan")
    z = [torch.empty_like(x) for x in a]
    assert status(lambda: B.dacp_syev_batched(ctx, a, z, noalloc=noalloc)) == -7
