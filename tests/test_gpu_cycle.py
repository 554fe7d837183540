"""The multigrid cycle on the GPU (coarse levels as two products each, the dense solve taking the
last restriction) against the same cycle written with the hierarchy's operators and
prolongators in numpy: PCG iteration counts on two to four levels, triangles and tetrahedra."""
import ctypes

import numpy as np
import pytest
import scipy.sparse as sp
import torch

pytestmark = pytest.mark.gpu

from gpu_util import make_pair  # noqa: E402


def _matrix(s, level, which):
    n, m, nnz = (ctypes.c_int64() for _ in range(3))
    arg = [s._h, level, which, ctypes.byref(n), ctypes.byref(m), ctypes.byref(nnz)]
    assert s._lib.dfdg_debug_multigrid_matrix(*arg, None, None, None) == 0
    ptr, col, val = np.zeros(n.value + 1, np.int64), np.zeros(nnz.value, np.int32), np.zeros(nnz.value)
    assert s._lib.dfdg_debug_multigrid_matrix(*arg, *(a.ctypes.data_as(ctypes.c_void_p) for a in (ptr, col, val))) == 0
    return sp.csr_matrix((val, col, ptr), shape=(n.value, m.value))


def _cycle(s):
    L = ctypes.c_int()
    rows, nnz, rho = np.zeros(16, np.int64), np.zeros(16, np.int64), np.zeros(16)
    assert s._lib.dfdg_debug_multigrid(s._h, 16, ctypes.byref(L), *(a.ctypes.data_as(ctypes.c_void_p)
                                                                    for a in (rows, nnz, rho))) == 0
    L = L.value
    A = [_matrix(s, l, 0) for l in range(L)]
    P = [_matrix(s, l, 1) for l in range(L - 1)]
    inv = _matrix(s, L - 1, 2).toarray()
    d = [1.0 / a.diagonal() for a in A]

    def apply(b, l=0):
        if l == L - 1:
            return inv @ b
        lmax = 1.05 * rho[l]
        lmin = lmax / (15.0 if l == 0 else 30.0)
        th, de = 0.5 * (lmax + lmin), 0.5 * (lmax - lmin)
        rho0 = de / th
        rho1 = 1.0 / (2.0 * th / de - rho0)
        c1, c2 = (rho1 * rho0, 2.0 * rho1 / de) if l == 0 else (0.0, 0.0)
        x1 = d[l] * b / th
        x = (1 + c1) * x1 + c2 * d[l] * (b - A[l] @ x1)
        x = x + P[l] @ apply(P[l].T @ (b - A[l] @ x), l + 1)
        e = d[l] * (b - A[l] @ x) / th
        x = x + e
        return x + c1 * e + c2 * d[l] * (b - A[l] @ x)

    return A[0], apply, L


def _pcg(A, M, g, rtol):
    x, r = np.zeros_like(g), g.copy()
    z = M(r)
    p, rz, it = z, r @ z, 0
    while np.linalg.norm(r) > rtol * np.linalg.norm(g):
        q = A @ p
        a = rz / (p @ q)
        x, r = x + a * p, r - a * q
        z = M(r)
        rz, old = r @ z, rz
        p, it = z + (rz / old) * p, it + 1
    return it


@pytest.mark.parametrize("mg_fp32", [False, True])
@pytest.mark.parametrize("dim,N,k,levels", [(2, 20, 2, 2), (2, 64, 2, 3), (2, 100, 3, 3), (3, 10, 1, 2), (3, 16, 2, 3)])
def test_iterations_equal_the_cycle_written_out(dim, N, k, levels, mg_fp32):
    """The same preconditioner up to rounding (FP16 values of S in an FP32 cycle: 5e-4 of each)
    takes the same iterations, within one."""
    rtol = 1e-9
    _, s, _, _ = make_pair(N, k, dim=dim, oracle=False, precond="amg", mg_fp32=mg_fp32, cg_rtol=rtol, facet_blocks=64)
    A, M, L = _cycle(s)
    assert L >= levels
    F = torch.randn(s.n_broken, generator=torch.Generator().manual_seed(N), dtype=torch.float64).to(s.device)
    lam = s.new_vector("lambda")
    _, info = s.mass_solve(F, lam=lam)
    g = A @ lam.cpu().numpy()
    its = _pcg(A, M, g, rtol)
    print(dim, N, k, "levels", L, "iterations", info.iterations, its, flush=True)
    assert abs(info.iterations - its) <= 1


@pytest.mark.parametrize("kw,tol", [(dict(mg_fp32=False), 1e-10), (dict(mg_fp32=True, mg_fine_fp16=False), 1e-4),
                                    (dict(mg_fp32=True), 1e-2)], ids=["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("dim,N,k,mesh", [(2, 37, 1, {}), (2, 21, 2, dict(walls=True)), (2, 15, 3, dict(inout=True)),
                                          (2, 24, 2, dict(mg_fine_smooth=3)), (3, 7, 1, dict(inout=True)),
                                          (3, 6, 2, dict(walls=True))])
def test_one_cycle_equals_the_cycle_written_out(dim, N, k, mesh, kw, tol):
    """One cycle on a random vector: the rounding of FP64 and FP32 (1e-16 and 6e-8 a step, times
    the coarse operator's condition, some 1e3) or of the FP16 values (5e-4 each)."""
    _, s, _, _ = make_pair(N, k, dim=dim, oracle=False, precond="amg", facet_blocks=64, **mesh, **kw)
    _, M, L = _cycle(s)
    assert L >= 2
    b = torch.randn(s.n_lambda, generator=torch.Generator().manual_seed(N), dtype=torch.float64)
    db, dz = b.to(s.device), s.new_vector("lambda")
    assert s._lib.dfdg_debug_vcycle(s._h, ctypes.c_void_p(db.data_ptr()), ctypes.c_void_p(dz.data_ptr())) == 0
    z = M(b.numpy())
    err = np.linalg.norm(dz.cpu().numpy() - z) / np.linalg.norm(z)
    print(dim, N, k, mesh, kw, "levels", L, err, flush=True)
    assert err < tol
