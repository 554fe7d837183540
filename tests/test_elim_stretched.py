"""Meshes of thin elements: the elimination's inverse in FP32 serves while the facet matrix,
scaled by its diagonal, is conditioned below 1e9 or so; well before that, a context takes the multigrid
cycle, which still converges there."""
import ctypes

import numpy as np
import pytest
import torch

from inputs import (channel_kuhn_cube, channel_split_square, distort_split_square, inout_split_square,
                    outflow_at_right, periodic_kuhn_cube, periodic_split_square)

lib_mod = pytest.importorskip("paper_1808_04669_amd.dfdg")


def _stretched(gen, N, aspect, axis=0):
    xyz, per = gen(N, "morton", 0)
    xyz, per = xyz.copy(), np.array(per, float)
    xyz[..., axis] *= aspect
    per[axis] *= aspect
    return xyz, per


def _layers(N, ratio):
    """Channel whose rows grow by a constant factor from the walls, by `ratio` in all."""
    xyz, per = channel_split_square(N, "morton", 0)
    h = ratio ** (np.minimum(np.arange(N), N - 1 - np.arange(N)) * 2.0 / N)
    y = np.concatenate([[0], np.cumsum(h)]) / h.sum()
    xyz = xyz.copy()
    xyz[..., 1] = y[np.rint(xyz[..., 1] * N).astype(int)]
    return xyz, np.array(per, float)


def _takes_elimination(xyz, per, k, outflow=None):
    lib = lib_mod.load_library()
    mesh = lib_mod.Mesh(xyz, per, outflow)
    p = lib_mod.Params()
    lib.dfdg_params_default(ctypes.byref(p))
    p.k, p.precond, p.elimination = k, 2, 2
    h = ctypes.c_void_p()
    rc = lib.dfdg_ctx_create(mesh._h, ctypes.byref(p), None, ctypes.byref(h))
    if rc == 0:
        lib.dfdg_ctx_destroy(h)
    assert rc in (0, -8)
    return rc == 0


@pytest.mark.parametrize("gen", [periodic_split_square, channel_split_square])
@pytest.mark.parametrize("axis", [0, 1])
def test_triangles(gen, axis):
    """Condition of the 24^2 BDM_2 system by dense eigenvalues of smaller ones, growing with
    (N aspect)^2: some 1e7 at an aspect of 100, 4e9 at 2000."""
    for aspect, takes in ((1, True), (20, True), (2000, False), (5000, False)):
        assert _takes_elimination(*_stretched(gen, 24, aspect, axis), 2) == takes, aspect


@pytest.mark.parametrize("gen", [periodic_kuhn_cube, channel_kuhn_cube])
@pytest.mark.parametrize("axis", [0, 2])
@pytest.mark.parametrize("N,k", [(6, 1), (5, 2)])
def test_tetrahedra(gen, axis, N, k):
    for aspect, takes in ((1, True), (3000, False), (10000, False)):
        assert _takes_elimination(*_stretched(gen, N, aspect, axis), k) == takes, aspect


def test_other_meshes():
    assert _takes_elimination(*_layers(24, 30), 2) and _takes_elimination(*_layers(24, 1000), 2)
    xyz, per = periodic_split_square(24, "morton", 0)
    assert _takes_elimination(distort_split_square(xyz, per, 24, 0.2, seed=3), per, 2)
    xyz, per = inout_split_square(24, "morton", 0)
    assert _takes_elimination(xyz, per, 2, outflow_at_right)
    xyz, per = _stretched(inout_split_square, 24, 4000, 0)
    assert not _takes_elimination(xyz, per, 2, lambda x: x[:, 0] > 3999.9)


@pytest.mark.gpu
@pytest.mark.parametrize("gen,aspect,rtol", [(periodic_split_square, 2000, 1e-10), (channel_split_square, 1000, 1e-10),
                                             (periodic_split_square, 30, 1e-12)])
def test_stretched_meshes_converge(gen, aspect, rtol):
    """The cycle's counts by a copy in numpy: 125, 221 and 135 to these tolerances."""
    s = lib_mod.Solver(*_stretched(gen, 24, aspect), 2, precond="amg", cg_rtol=rtol, cg_maxit=4000)
    F = torch.randn(s.n_broken, generator=torch.Generator().manual_seed(5), dtype=torch.float64).to(s.device)
    U, info = s.mass_solve(F)
    print(gen.__name__, aspect, info.iterations, info.rel_residual, flush=True)
    assert info.status == 0 and info.rel_residual <= rtol and bool(torch.isfinite(U).all())
