"""The largest systems that take the block elimination (interfaces of some 9000 unknowns, cell
fronts above 1000), against the multigrid cycle, and the sizes just above that fall back to it."""
import ctypes

import pytest
import torch

from inputs import periodic_kuhn_cube, periodic_split_square

lib_mod = pytest.importorskip("paper_1808_04669_amd.dfdg")


@pytest.mark.parametrize("dim,N,k,takes", [(3, 11, 1, True), (3, 12, 1, False), (3, 8, 2, True), (3, 9, 2, False),
                                           (2, 73, 1, True), (2, 74, 1, False), (2, 52, 3, True), (2, 53, 3, False)])
def test_limits(dim, N, k, takes):
    """2D: E (k + 1) up to 32768 multipliers.  3D: the matrices, up to 128 Mi values, end it first."""
    lib = lib_mod.load_library()
    mesh = lib_mod.Mesh(*(periodic_split_square if dim == 2 else periodic_kuhn_cube)(N, "morton"))
    p = lib_mod.Params()
    lib.dfdg_params_default(ctypes.byref(p))
    p.k, p.precond, p.elimination = k, 2, 2
    h = ctypes.c_void_p()
    rc = lib.dfdg_ctx_create(mesh._h, ctypes.byref(p), None, ctypes.byref(h))
    assert rc == (0 if takes else -8)
    if rc == 0:
        lib.dfdg_ctx_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("dim,N,k,kw", [(3, 11, 1, {}), (3, 10, 1, dict(walls=True, order="random")), (3, 8, 2, {}),
                                        (3, 7, 2, dict(inout=True, order="random")), (2, 73, 1, {}),
                                        (2, 52, 3, dict(order="random"))])
def test_largest_equal_multigrid(dim, N, k, kw):
    """Solves to 1e-12 of one right-hand side: velocities within 1e-9 (the residual times the square
    root of the condition, below 1e6 here)."""
    from gpu_util import make_pair
    out = []
    for elim in (True, False):
        _, s, _, _ = make_pair(N, k, dim=dim, oracle=False, cg_rtol=1e-12, precond="amg", elimination=elim, **kw)
        F = torch.randn(s.n_broken, generator=torch.Generator().manual_seed(3), dtype=torch.float64).to(s.device)
        U, info = s.mass_solve(F)
        assert info.status == 0 and info.rel_residual <= 1e-12
        out.append((U, info.iterations))
        del s
    print(dim, N, k, kw, "iterations", out[0][1], out[1][1], flush=True)
    assert out[0][1] <= 4 < out[1][1]
    assert (out[0][0] - out[1][0]).norm() <= 1e-9 * out[1][0].norm()
