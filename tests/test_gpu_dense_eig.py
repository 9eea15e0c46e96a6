"""Dense symmetric eigensolver at the sizes where its stages change (MI355X).

Leaves of the divide and conquer hold at most 32 rows, its products use 64 x 64 tiles, and blocks are
halved unevenly; matrices with clusters, exact splits and zeros exercise the deflation.  Against
numpy's FP64 eigensolver; an error of a backward stable method is a modest multiple of
n eps ||A||, taken here as 20 (eigenvalues, residuals) and 20 n eps (orthogonality).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2011_02107_amd import binding as B  # noqa: E402

pytestmark = pytest.mark.gpu

EPS = 2.220446049250313e-16


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    c.tune("dc", 1)
    yield c
    torch.cuda.synchronize()
    c.close()


def matrix(kind, n):
    rng = np.random.default_rng(n)
    q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    if kind == "random":
        a = rng.standard_normal((n, n))
        return 0.5 * (a + a.T)
    if kind == "low_rank":  # most eigenvalues at the rounding level, as in an oversampled overlap matrix
        r = max(1, n // 3)
        lam = np.concatenate([np.zeros(n - r), rng.uniform(0.1, 3.0, r)])
    elif kind == "clusters":  # a few values, each many times
        lam = rng.integers(-2, 3, n).astype(float)
    elif kind == "graded":
        lam = 10.0 ** rng.uniform(-14, 0, n)
    elif kind == "diagonal":
        return np.diag(rng.standard_normal(n))
    elif kind == "tridiagonal":  # with exact splits
        e = rng.standard_normal(n - 1)
        e[::7] = 0.0
        return np.diag(rng.standard_normal(n)) + np.diag(e, 1) + np.diag(e, -1)
    else:
        return np.zeros((n, n))
    a = (q * lam) @ q.T
    return 0.5 * (a + a.T)


def check(ctx, a):
    n = a.shape[0]
    A = torch.as_tensor(a, dtype=torch.float64, device="cuda:0").contiguous()
    Z = torch.empty_like(A)
    w = B.dacp_syev(ctx, A, Z)
    z = Z.cpu().numpy()
    norm = np.abs(np.linalg.eigvalsh(a)).max()
    assert np.abs(w - np.linalg.eigvalsh(a)).max() <= 20 * n * EPS * norm
    assert np.abs(z @ z.T - np.eye(n)).max() <= 20 * n * EPS
    assert np.abs(z @ a - w[:, None] * z).max() <= 20 * n * EPS * norm


@pytest.mark.parametrize("n", [2, 3, 5, 31, 32, 33, 63, 64, 65, 66, 129, 257, 513, 1030, 2047, 2049])
def test_syev_sizes(ctx, n):
    check(ctx, matrix("random", n))


@pytest.mark.parametrize("kind", ["low_rank", "clusters", "graded", "diagonal", "tridiagonal", "zero"])
@pytest.mark.parametrize("n", [40, 97, 300, 777])
def test_syev_deflation(ctx, kind, n):
    check(ctx, matrix(kind, n))


@pytest.mark.parametrize("n", [2050, 2561, 3072, 3073])
def test_syev_largest_on_chip(ctx, n):
    """Beyond 2048 rows the reflectors are applied a block at a time through the GEMM; beyond 3072 the
    matrix stays in memory.  A = Q diag(lam) Q^T by one reflector Q, so that the spectrum is known."""
    rng = np.random.default_rng(n)
    lam = np.sort(rng.standard_normal(n))
    u = rng.standard_normal(n)
    u *= np.sqrt(2.0) / np.linalg.norm(u)
    a = np.diag(lam) - np.outer(u, u * lam) - np.outer(u * lam, u) + (u @ (u * lam)) * np.outer(u, u)
    a = 0.5 * (a + a.T)
    A = torch.as_tensor(a, device="cuda:0").contiguous()
    Z = torch.empty_like(A)
    w = B.dacp_syev(ctx, A.clone(), Z)
    norm = np.abs(lam).max()
    wt = torch.as_tensor(w, device="cuda:0")
    eye = torch.eye(n, dtype=torch.float64, device="cuda:0")
    assert np.abs(w - lam).max() <= 20 * n * EPS * norm
    assert float((Z @ Z.T - eye).abs().max()) <= 20 * n * EPS
    assert float((Z @ A - wt[:, None] * Z).abs().max()) <= 20 * n * EPS * norm
