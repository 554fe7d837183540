"""GPU checks of the matrix-free products of the facet system on tetrahedra (element pass with
the two sides of each face, Jacobi update that sums them): the products, the solves and the
multiplier against the assembled S, with closed, inflow and outflow boundaries, point and
facet-block Jacobi and the multigrid cycle, on grids with fewer and more blocks than elements
fill."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from gpu_util import make_pair  # noqa: E402


@pytest.mark.parametrize("N,k,precond,kw", [
    (2, 1, "jacobi", {}), (3, 2, "block_jacobi", {}), (4, 1, "block_jacobi", dict(walls=True)),
    (3, 2, "jacobi", dict(inout=True)), (5, 2, "jacobi", dict(order="random", facet_blocks=3)),
    (6, 1, "amg", dict(walls=True, facet_blocks=7)), (4, 2, "amg", dict(inout=True, facet_blocks=1024)),
    (12, 2, "jacobi", {}),
])
def test_element_products_equal_the_assembled_matrix(N, k, precond, kw):
    """Both forms of S agree to rounding (1e-15 of the row sums), so solves to 1e-12 take the
    same iterations within one; a velocity differs by the two residuals over the square root
    of the smallest eigenvalue, far below 1e-9 of it."""
    out = []
    g = torch.Generator(device="cpu").manual_seed(5)
    for mf in (False, True):
        _, s, _, _ = make_pair(N, k, dim=3, oracle=False, cg_rtol=1e-12, precond=precond, matrix_free=mf, **kw)
        if not out:
            F = torch.randn(s.n_broken, generator=g, dtype=torch.float64).to(s.device)
        lam = s.new_vector("lambda")
        U, info = s.mass_solve(F, lam=lam)
        assert info.status == 0 and info.rel_residual <= 1e-12
        out.append((U, lam, info.iterations))
    (U0, l0, i0), (U1, l1, i1) = out
    print(N, k, precond, kw, "iterations", i0, i1, flush=True)
    assert abs(i0 - i1) <= 1
    assert (U1 - U0).norm() <= 1e-9 * U0.norm() and (l1 - l0).norm() <= 1e-8 * l0.norm()


def test_large_meshes_take_the_element_products():
    """18^3 (34992 elements, above the line): the products asked for and the default ones give
    the same bits."""
    out = []
    g = torch.Generator(device="cpu").manual_seed(5)
    for mf in (False, True):
        _, s, _, _ = make_pair(18, 1, dim=3, oracle=False, cg_rtol=1e-10, matrix_free=mf)
        F = torch.randn(s.n_broken, generator=torch.Generator(device="cpu").manual_seed(5),
                        dtype=torch.float64).to(s.device)
        out.append(s.mass_solve(F)[0])
    assert torch.equal(out[0], out[1])
