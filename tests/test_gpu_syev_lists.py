"""Lists of dense eigenproblems that do not go in one round (MI355X): less memory than the whole list's scratch takes, more rows than the compute units hold at once.

Bounds as for one matrix: a backward stable method's error is a modest multiple of n eps ||A||, taken as 20.
"""
import pytest

torch = pytest.importorskip("torch")

from paper_2011_02107_amd import binding as B  # noqa: E402

pytestmark = pytest.mark.gpu

EPS = 2.220446049250313e-16
DEV = "cuda:0"
MIB = 1 << 20


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def symmetric(count, n, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    a = torch.randn(count, n, n, generator=g, device=DEV, dtype=torch.float64)
    return (a + a.transpose(1, 2)).contiguous()


def check(a, w, z):
    """Residuals and orthogonality of every matrix of a (count, n, n), the eigenvectors the rows of z."""
    n = a.shape[1]
    norm = w.abs().amax(dim=1)
    assert bool((w[:, 1:] >= w[:, :-1]).all())
    eye = torch.eye(n, device=DEV, dtype=torch.float64)
    for i0 in range(0, a.shape[0], 4096):
        s = slice(i0, i0 + 4096)
        zt = z[s].transpose(1, 2).contiguous()
        assert (torch.bmm(z[s], zt) - eye).abs().max().item() <= 20 * n * EPS
        r = (torch.bmm(z[s], a[s]) - w[s][:, :, None] * z[s]).abs().amax(dim=(1, 2))
        assert bool((r <= 20 * n * EPS * norm[s]).all())
        tr = torch.diagonal(a[s], dim1=1, dim2=2).sum(dim=1)  # every eigenvalue once
        assert bool(((w[s].sum(dim=1) - tr).abs() <= 20 * n * n * EPS * norm[s]).all())


def solve(ctx, a):
    work, z = a.clone(), torch.empty_like(a)
    w = B.dacp_syev_batched(ctx, list(work), list(z))
    return torch.as_tensor([list(x) for x in w], dtype=torch.float64, device=DEV), z


def test_less_memory_than_the_scratch(ctx):
    a = symmetric(64, 512, 2)
    work, z = a.clone(), torch.empty_like(a)
    w = B.dacp_syev_batched(ctx, list(work), list(z))  # loads the kernels
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    work.copy_(a)
    z.zero_()
    filler, left = [], 400
    try:
        for _ in range(8):
            more = torch.cuda.mem_get_info()[0] - left * MIB
            if more < 4 * MIB:
                break
            filler.append(torch.empty(more, dtype=torch.uint8, device=DEV))
        assert torch.cuda.mem_get_info()[0] <= (left + 4) * MIB
        w = B.dacp_syev_batched(ctx, list(work), list(z))
        torch.cuda.synchronize()
    finally:
        del filler
        torch.cuda.empty_cache()
    check(a, torch.as_tensor([list(x) for x in w], dtype=torch.float64, device=DEV), z)


@pytest.mark.parametrize("count,n", [(4, 1000), (3, 1500), (3, 2047), (9, 1000), (5, 1025), (12, 700), (30, 300)])
def test_rows_past_the_compute_units(ctx, count, n):
    """A single matrix takes few rows a workgroup; lists take the larger shape of their row length, and
    more than one cooperative launch where even that is not enough."""
    a = symmetric(count, n, 3)
    w, z = solve(ctx, a)
    check(a, w, z)
