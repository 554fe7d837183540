"""The bytes dfdg_time_kernel reports, counted here from the kernels' arrays: each array once."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import make_pair  # noqa: E402


@pytest.mark.parametrize("k", [1, 2])
def test_jacobi_update(k):
    """p, S p, x, r, D^{-1} in, x, r, z out; behind element products S p as its two sides."""
    for mf, vectors in ((False, 8), (True, 9)):
        _, s, _, _ = make_pair(4, k, dim=3, oracle=False, matrix_free=mf)
        assert s.time_kernel(1, reps=1)[1] == 8 * vectors * s.n_lambda


@pytest.mark.parametrize("dim,N,k,kw", [(2, 20, 2, {}), (2, 20, 1, dict(mg_fp32=False)), (2, 20, 2, dict(mg_fine_fp16=False)),
                                        (3, 4, 2, {})])
def test_cycle_of_two_levels(dim, N, k, kw):
    _, s, _, _ = make_pair(N, k, dim=dim, oracle=False, precond="amg", elimination=False, **kw)
    assert len(s.mg_levels()) == 2
    n, nc = s.mg_levels()
    E, NF, NS = s.E, s.n_lambda // s.E, 5 if dim == 2 else 7
    fp32, half = kw.get("mg_fp32", True), kw.get("mg_fp32", True) and kw.get("mg_fine_fp16", True)
    v = 4 if fp32 else 8
    P = s.mg_matrix(0, 1).tocoo()
    pairs = len(np.unique(P.row // NF * np.int64(nc) + P.col))  # columns of the facets
    widest = np.bincount(np.unique(P.row // NF * np.int64(nc) + P.col) // nc).max()
    S = E * NS * 4 + ((E * ((NS * NF * NF + 1) // 2) * 4) if half else E * NS * NF * NF * v)
    if half and widest <= 16:  # prolongation, restriction
        xfer = pairs * (2 + 2 * NF) + pairs * (4 + 4 * ((NF + 1) // 2))
    else:
        xfer = 2 * pairs * (4 + v * NF)
    assert s.time_kernel(4, reps=1)[1] == 4 * S + 17 * n * v + xfer + (2 * n + 2 * nc) * v + nc * nc * v
