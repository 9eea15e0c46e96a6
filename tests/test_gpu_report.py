"""Fields of the report that name the evolution's column groups (MI355X)."""
import pytest

torch = pytest.importorskip("torch")

from paper_2011_02107_amd import binding as B  # noqa: E402
from paper_2011_02107_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,b,group,moment_mode,want", [(10, 6, 0, 0, 6), (10, 6, 2, 0, 2), (15, 16, 0, 0, 8), (15, 16, 0, 2, 8),
                                                        (15, 12, 4, 1, 4)])
def test_evolution_group_is_the_column_group_width(L, b, group, moment_mode, want):
    """The width asked for, or 8 columns from 15 spins on, however many groups share a launch."""
    ctx = B.Context(0)
    ham = B.dacp_build_hamiltonian(ctx, L, inputs.ising_chain(L))
    _, _, rep, _ = B.dacp_central_eigs(ctx, ham, 24, B.default_opts(b=b, seed=1, group=group, moment_mode=moment_mode))
    assert rep["evol_group"] == want
    ham.close()
    ctx.close()
