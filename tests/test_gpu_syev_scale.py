"""The dense eigensolvers on matrices whose scale is far from 1 (MI355X): the products of the tridiagonalisation and of
the secular equation square and cube the entries, which may not leave the range of a double."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2011_02107_amd import binding as B  # noqa: E402

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("power", [-498, -460, -350, 350, 460, 498])
@pytest.mark.parametrize("n", [20, 200, 700])
def test_scale(ctx, n, power):
    a = np.random.default_rng(n).standard_normal((n, n))
    a = (a + a.T) / 2
    ref = np.linalg.eigvalsh(a)
    tol = 20 * n * EPS * np.abs(ref).max()
    m = torch.as_tensor(np.ldexp(a, power), device="cuda:0").contiguous()  # a power of two: exact
    z = torch.empty_like(m)
    batch = [torch.empty_like(m), torch.empty(33, 33, device="cuda:0", dtype=torch.float64)]
    small = torch.diag(torch.arange(33, device="cuda:0", dtype=torch.float64))  # its own scale stays 1
    found = [B.dacp_syev(ctx, m.clone(), z), B.dacp_syev(ctx, m.clone(), None)]
    w = B.dacp_syev_batched(ctx, [m.clone(), small], batch)
    np.testing.assert_allclose(w[1], np.arange(33.0), rtol=0, atol=20 * 33 * EPS * 32)
    for got in found + [w[0]]:
        np.testing.assert_allclose(np.ldexp(got, -power), ref, rtol=0, atol=tol)
    for vecs in (z, batch[0]):  # row e holds eigenvector e
        v = vecs.cpu().numpy()
        assert np.abs(v @ v.T - np.eye(n)).max() <= 20 * n * EPS
        assert np.abs(v @ a - ref[:, None] * v).max() <= tol
