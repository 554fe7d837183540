"""GPU checks of point-Jacobi iterations in one launch (update and product in one kernel, beta
from a predicted residual norm) against the two-kernel form, which a grid smaller than the
rows selects: triangles and tetrahedra, blocks of 64, 128 and 256 threads, closed, inflow and
outflow boundaries, the iteration limit, a zero right-hand side, eager launches."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from gpu_util import make_pair  # noqa: E402


def _pair(N, k, dim, **kw):
    # E / 256 blocks, less one, select the two kernels
    blocks = (3 * N * N // 256) if dim == 2 else (12 * N ** 3 // 256)
    out = []
    for fb in (0, max(1, blocks - 1)):
        _, s, _, _ = make_pair(N, k, dim=dim, oracle=False, precond="jacobi", facet_blocks=fb, **kw)
        out.append(s)
    return out


def _rhs(s, seed=3):
    return torch.randn(s.n_broken, generator=torch.Generator().manual_seed(seed), dtype=torch.float64).to(s.device)


@pytest.mark.parametrize("dim,N,k,kw", [
    (2, 10, 1, {}), (2, 24, 3, dict(walls=True)), (2, 25, 2, dict(inout=True)), (2, 75, 2, dict(order="random")),
    (2, 150, 1, {}), (2, 32, 2, dict(graphs=False)), (3, 5, 1, dict(inout=True)), (3, 5, 2, dict(walls=True)),
    (3, 9, 2, {}), (3, 13, 1, {}),
])
def test_one_launch_equals_two_kernels(dim, N, k, kw):
    """To 1e-11 of the residual both take the same iterations within one in fifty (a prediction
    differs from the norm by rounding), and the velocities agree far below 1e-8."""
    one, two = _pair(N, k, dim, cg_rtol=1e-11, **kw)
    F = _rhs(one)
    res = []
    for s in (one, two):
        lam = s.new_vector("lambda")
        U, info = s.mass_solve(F, lam=lam)
        assert info.status == 0 and info.rel_residual <= 1e-11
        res.append((U, info.iterations))
    print(dim, N, k, kw, "iterations", res[0][1], res[1][1], flush=True)
    assert abs(res[0][1] - res[1][1]) <= 1 + res[1][1] // 50
    assert (res[0][0] - res[1][0]).norm() <= 1e-8 * res[1][0].norm()


def test_iteration_limit_and_zero_right_hand_side():
    """A solve of n iterations converges with the limit n and stops as not converged with the
    limit n - 1, in both forms; a zero right-hand side takes no iterations."""
    from paper_1808_04669_amd import DfdgError
    for form in (0, 1):
        s = _pair(20, 2, 2, cg_rtol=1e-9)[form]
        F = _rhs(s)
        n = s.mass_solve(F)[1].iterations
        assert _pair(20, 2, 2, cg_rtol=1e-9, cg_maxit=n)[form].mass_solve(F)[1].iterations == n
        with pytest.raises(DfdgError, match="converge"):
            _pair(20, 2, 2, cg_rtol=1e-9, cg_maxit=n - 1)[form].mass_solve(F)
        U, info = s.mass_solve(torch.zeros_like(F))
        assert info.status == 0 and info.iterations == 0 and U.abs().max() == 0
