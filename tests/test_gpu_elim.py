"""GPU checks of the block elimination that preconditions the facet solves of small meshes
(cells and their interface, an exact solve in FP32): the same velocities as the multigrid
cycle's solves (facet_blocks set: the kernel-per-phase cycle of any size), in a few
iterations, at the smallest and largest systems that take it, with partial tiles and pivot
blocks, on every kind of boundary and numbering."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from gpu_util import make_pair, rel_l2, transfer  # noqa: E402
from inputs import RandomStreamField  # noqa: E402

CASES = [
    (2, 19, 1, {}), (2, 14, 2, {}), (2, 11, 3, {}), (3, 4, 1, {}), (3, 3, 2, {}),  # just above the dense level
    (2, 23, 2, dict(order="random", distort=0.15)), (2, 17, 3, dict(walls=True)), (2, 30, 1, dict(inout=True)),
    (3, 5, 1, dict(walls=True, order="random")), (3, 4, 2, dict(inout=True)), (2, 20, 2, dict(local_space="fe4")),
    (2, 60, 2, {}), (2, 48, 3, dict(distort=0.1)), (3, 7, 2, {}),  # the largest of its range
]


@pytest.mark.parametrize("dim,N,k,kw", CASES)
def test_elimination_equals_multigrid(dim, N, k, kw):
    """Solves to 1e-12 of one right-hand side: the velocity error of each is the residual
    times at most the square root of the facet system's condition (below 1e6 here) over the
    right-hand side's own share, so 1e-9 bounds their difference."""
    sol = []
    g = torch.Generator(device="cpu").manual_seed(3)
    for blocks in (0, 1024):
        _, s, _, _ = make_pair(N, k, dim=dim, oracle=False, cg_rtol=1e-12, precond="amg", facet_blocks=blocks, **kw)
        if not sol:
            F = torch.randn(s.n_broken, generator=g, dtype=torch.float64).to(s.device)
        U, info = s.mass_solve(F)
        assert info.status == 0 and info.rel_residual <= 1e-12
        sol.append((U, info.iterations))
        if blocks == 0:  # warm start, and the multiplier returned
            lam = s.new_vector("lambda")
            s.mass_solve(F, lam=lam)
            V, i2 = s.mass_solve(F, lam=lam)
            assert i2.iterations <= 1 and (V - U).norm() <= 1e-9 * U.norm()
    print(dim, N, k, kw, "iterations", [i for _, i in sol], flush=True)
    assert sol[0][1] <= 4 < sol[1][1]
    assert (sol[0][0] - sol[1][0]).norm() <= 1e-9 * sol[1][0].norm()


def test_elimination_steps_against_the_oracle():
    """Three TVD-RK3 steps on a distorted 15 x 15 mesh (the elimination's smallest range)
    against the CPU oracle, and the same bits from captured and from single launches."""
    out = []
    for graphs in (False, True):
        orc, s, _, _ = make_pair(15, 2, nu=1e-3, distort=0.1, oracle=True, precond="amg", extrapolate="project",
                                 cg_rtol=1e-13, graphs=graphs)
        Uo = orc.project(RandomStreamField(seed=3, kmax=3))
        U = transfer(orc, Uo, s)
        for _ in range(3):
            info = s.rk3_step(U, 0.002)
            assert info.status == 0 and max(info.iterations) <= 4
            Uo = orc.rk3_step(Uo, 0.002)
        assert rel_l2(orc, s, U, Uo) < 1e-10
        out.append(U)
    assert torch.equal(out[0], out[1]) and np.isfinite(out[0].sum().item())
