"""The hierarchy's derived matrices: the products a debug entry forms on request (CPU), and the last
restriction multiplied into the dense solve on the GPU, through whole cycles of three levels."""
import ctypes

import numpy as np
import pytest
import scipy.sparse as sp
import torch

from inputs import periodic_split_square

lib_mod = pytest.importorskip("paper_1808_04669_amd.dfdg")


def test_products_on_request():
    lib = lib_mod.load_library()
    mesh = lib_mod.Mesh(*periodic_split_square(64, "morton"))
    p = lib_mod.Params()
    lib.dfdg_params_default(ctypes.byref(p))
    p.k, p.precond = 2, 2
    h = ctypes.c_void_p()
    assert lib.dfdg_ctx_create(mesh._h, ctypes.byref(p), None, ctypes.byref(h)) == 0

    def matrix(level, which):
        n, m, nnz = (ctypes.c_int64() for _ in range(3))
        arg = [h, level, which, ctypes.byref(n), ctypes.byref(m), ctypes.byref(nnz)]
        rc = lib.dfdg_debug_multigrid_matrix(*arg, None, None, None)
        if rc:
            return rc
        ptr, col, val = np.zeros(n.value + 1, np.int64), np.zeros(nnz.value, np.int32), np.zeros(nnz.value)
        assert lib.dfdg_debug_multigrid_matrix(*arg, *(a.ctypes.data_as(ctypes.c_void_p) for a in (ptr, col, val))) == 0
        return sp.csr_matrix((val, col, ptr), shape=(n.value, m.value))

    A, P = matrix(1, 0), matrix(1, 1)
    assert abs(matrix(1, 3) - A @ P).max() < 1e-13 * abs(A).max()
    assert abs(matrix(1, 4) - (A @ P).T).max() < 1e-13 * abs(A).max()
    assert matrix(0, 3) == -1 and matrix(0, 4) == -1  # level 0 has none
    lib.dfdg_ctx_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("kw,tol", [(dict(mg_fp32=False), 1e-10), (dict(mg_fine_fp16=False), 1e-4)], ids=["fp64", "fp32"])
@pytest.mark.parametrize("dim,N,k", [(2, 64, 2), (2, 75, 1), (2, 90, 2), (3, 10, 1)])
def test_cycle_with_the_folded_restriction(dim, N, k, kw, tol):
    """One cycle on a random vector against the same cycle in numpy: rounding (1e-16 or 6e-8 a step)
    times the coarse operator's condition, some 1e3."""
    from gpu_util import make_pair
    from test_gpu_cycle import _cycle
    _, s, _, _ = make_pair(N, k, dim=dim, oracle=False, precond="amg", elimination=False, **kw)
    _, M, L = _cycle(s)
    assert L >= 3
    b = torch.randn(s.n_lambda, generator=torch.Generator().manual_seed(N), dtype=torch.float64)
    z = M(b.numpy())
    err = np.linalg.norm(s.vcycle(b.to(s.device)).cpu().numpy() - z) / np.linalg.norm(z)
    print(dim, N, k, kw, s.mg_levels(), err, flush=True)
    assert err < tol
