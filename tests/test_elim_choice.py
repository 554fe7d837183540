"""The choice between the block elimination and the multigrid cycle (dfdg_params.elimination),
and facet_blocks as a launch shape: a cap that the default grid does not reach changes
nothing, one that it exceeds leaves the chosen preconditioner alone."""
import ctypes

import pytest
import torch

from inputs import periodic_split_square

lib_mod = pytest.importorskip("paper_1808_04669_amd.dfdg")


def _create(N, **kw):
    lib = lib_mod.load_library()
    mesh = lib_mod.Mesh(*periodic_split_square(N, "morton"))
    p = lib_mod.Params()
    lib.dfdg_params_default(ctypes.byref(p))
    for k, v in kw.items():
        setattr(p, k, v)
    h = ctypes.c_void_p()
    rc = lib.dfdg_ctx_create(mesh._h, ctypes.byref(p), None, ctypes.byref(h))
    if rc == 0:
        lib.dfdg_ctx_destroy(h)
    return rc


@pytest.mark.parametrize("N,kw,rc", [
    (19, dict(elimination=0), 0), (19, dict(elimination=1), 0), (19, dict(elimination=2), 0),
    (19, dict(elimination=2, facet_blocks=3), 0), (19, dict(elimination=2, mg_fp32=0), -8),
    (19, dict(elimination=2, precision=1), 0), (19, dict(elimination=2, precision=1, mixed_solver=0), -8),
    (19, dict(elimination=2, precond=0), -8), (8, dict(elimination=2), -8),  # 8^2 BDM_2: one dense level
    (64, dict(elimination=2), -8), (19, dict(elimination=3), -1), (19, dict(elimination=-1), -1),
])
def test_what_a_context_accepts(N, kw, rc):
    assert _create(N, **dict(dict(k=2, precond=2), **kw)) == rc


def _solve(**kw):
    from gpu_util import make_pair
    _, s, _, _ = make_pair(20, 2, oracle=False, cg_rtol=1e-12, **kw)
    F = torch.randn(s.n_broken, generator=torch.Generator().manual_seed(4), dtype=torch.float64).to(s.device)
    U, info = s.mass_solve(F)
    assert info.status == 0
    return U, info.iterations


@pytest.mark.gpu
def test_facet_blocks_leaves_the_preconditioner_alone():
    """Solves to 1e-12 of the right-hand side: 1e-9 of the velocity (see test_gpu_elim)."""
    U, n = _solve(precond="amg")
    for blocks in (0, 1, 7, 1024):
        V, m = _solve(precond="amg", facet_blocks=blocks, elimination=True)
        assert abs(m - n) <= 1 and n <= 4 and (V - U).norm() <= 1e-9 * U.norm()
    C, c = _solve(precond="amg", elimination=False)
    assert c > 4 and (C - U).norm() <= 1e-9 * U.norm()
    assert torch.equal(C, _solve(precond="amg", facet_blocks=1024)[0])
    assert torch.equal(C, _solve(precond="amg", facet_blocks=1024, elimination=False)[0])


@pytest.mark.gpu
def test_a_cap_above_the_grid_changes_nothing():
    for precond in ("jacobi", "block_jacobi"):
        assert torch.equal(_solve(precond=precond)[0], _solve(precond=precond, facet_blocks=1024)[0])
