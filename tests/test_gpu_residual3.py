"""The tetrahedral residual on a discontinuous random field next to outflow, inflow and wall
boundaries: own and neighbour traces in modes, the upwind choice at every face point, outflow
with backflow, elements that fill no whole block."""
import numpy as np
import pytest

from inputs import eval_broken_poly_3d, random_broken_poly_3d
from oracle.quadrature import tet_rule

pytestmark = pytest.mark.gpu

from gpu_util import broken_residual_on_oracle_basis, make_pair, values_to_lib  # noqa: E402


@pytest.mark.parametrize("kw", [dict(inout=True), dict(walls=True), {}], ids=["inout", "walls", "periodic"])
@pytest.mark.parametrize("k,N,nu", [(1, 2, 0.0), (1, 3, 0.03), (2, 2, 0.03), (2, 3, 0.0), (2, 4, 0.03)])
def test_broken_field_next_to_boundaries(k, N, nu, kw):
    """Entrywise to 1e-11 of the largest entry: sums of some 1e3 terms, each to 1e-15."""
    orc, s, _, _ = make_pair(N, k, nu=nu, order="random", seed=N, dim=3, **kw)
    coef = random_broken_poly_3d(s.T, k, seed=7 * k + N)
    U = values_to_lib(s, lambda pts: eval_broken_poly_3d(coef, pts))
    rule = tet_rule(2 * k)
    R_orc = orc.res.broken(orc.space.broken_project(eval_broken_poly_3d(coef, rule[0]), rule))
    R_gpu = broken_residual_on_oracle_basis(orc, s, s.residual(U))
    err = np.abs(R_gpu - R_orc).max() / np.abs(R_orc).max()
    print(k, N, nu, kw, err, flush=True)
    assert err < 1e-11
