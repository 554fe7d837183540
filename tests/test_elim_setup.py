"""Set-up of contexts that solve by elimination: no multigrid hierarchy is built for them unless a
debug entry point asks for it, and what those entry points return does not change."""
import ctypes
import time

import numpy as np
import pytest
import torch

from inputs import channel_split_square, periodic_kuhn_cube, periodic_split_square

lib_mod = pytest.importorskip("paper_1808_04669_amd.dfdg")


def _create(mesh, **kw):
    lib = lib_mod.load_library()
    p = lib_mod.Params()
    lib.dfdg_params_default(ctypes.byref(p))
    p.precond = 2
    for k, v in kw.items():
        setattr(p, k, v)
    h = ctypes.c_void_p()
    t = time.perf_counter()
    rc = lib.dfdg_ctx_create(mesh._h, ctypes.byref(p), None, ctypes.byref(h))
    return rc, h, time.perf_counter() - t


def _levels(h):
    lib = lib_mod.load_library()
    n = ctypes.c_int()
    rows, nnz, rho = np.zeros(16, np.int64), np.zeros(16, np.int64), np.zeros(16)
    assert lib.dfdg_debug_multigrid(h, 16, ctypes.byref(n), *(a.ctypes.data_as(ctypes.c_void_p)
                                                              for a in (rows, nnz, rho))) == 0
    return rows[:n.value].tolist(), nnz[:n.value].tolist(), rho[:n.value].tolist()


def test_no_hierarchy_at_creation():
    """The hierarchy is most of a small context's set-up (40 of 41 parts at 16^2 BDM_1): without
    it a context takes less than half the time."""
    lib = lib_mod.load_library()
    mesh = lib_mod.Mesh(*periodic_split_square(16, "morton"))
    best = {}
    for elim in (2, 1):
        for _ in range(5):
            rc, h, t = _create(mesh, k=1, elimination=elim)
            assert rc == 0
            best[elim] = min(t, best.get(elim, t))
            lib.dfdg_ctx_destroy(h)
    assert best[2] < 0.5 * best[1], best


@pytest.mark.parametrize("gen,N,k,stretch,several", [
    (periodic_split_square, 10, 2, 1, False), (periodic_split_square, 11, 2, 1, True),  # 900 and 1089 unknowns
    (channel_split_square, 16, 1, 30, False), (channel_split_square, 16, 2, 100, False),  # coarsening stalls: dense
    (channel_split_square, 16, 1, 3, True), (periodic_kuhn_cube, 3, 2, 1, True), (periodic_kuhn_cube, 2, 2, 1, False),
])
def test_levels_decide_as_before(gen, N, k, stretch, several):
    """The elimination serves where the multigrid has two levels or more; asked for its levels,
    such a context gives those of one that uses the cycle."""
    lib = lib_mod.load_library()
    xyz, per = gen(N, "morton", 0)
    xyz, per = xyz.copy(), np.array(per, float)
    xyz[..., 0] *= stretch
    per[0] *= stretch
    mesh = lib_mod.Mesh(xyz, per)
    rc, h, _ = _create(mesh, k=k, elimination=1)
    assert rc == 0
    cycle = _levels(h)
    lib.dfdg_ctx_destroy(h)
    assert (len(cycle[0]) >= 2) == several
    rc, h, _ = _create(mesh, k=k, elimination=2)
    assert rc == (0 if several else -8)
    if rc == 0:
        assert _levels(h) == cycle
        lib.dfdg_ctx_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("dim,N,k,kw", [(2, 20, 2, {}), (2, 20, 1, dict(precision="mixed")), (3, 4, 2, {})])
def test_debug_entries_of_the_cycle(dim, N, k, kw):
    """The same bits from a context that uses the cycle and from one that does not; the solves of
    the latter are left alone."""
    from gpu_util import make_pair
    out = []
    for elim in (False, True):
        _, s, _, _ = make_pair(N, k, dim=dim, oracle=False, precond="amg", elimination=elim, cg_rtol=1e-11, **kw)
        F = torch.randn(s.n_broken, generator=torch.Generator().manual_seed(2), dtype=torch.float64).to(s.device)
        b = torch.randn(s.n_lambda, generator=torch.Generator().manual_seed(3), dtype=torch.float64).to(s.device)
        U = s.mass_solve(F)[0].clone()
        z, z2 = s.vcycle(b), s.vcycle(b)
        ms, nbytes = s.time_kernel(4, reps=2)
        assert ms > 0 and torch.equal(z, z2) and torch.equal(s.mass_solve(F)[0], U)
        out.append((z, nbytes, s.mg_levels()))
    assert torch.equal(out[0][0], out[1][0]) and out[0][1:] == out[1][1:]


def test_workspace_without_the_scratch():
    """The factorisation's arrays (fronts, interface and panels in FP64, the element matrices) are
    no part of what a context keeps: that stays below half of the whole."""
    lib = lib_mod.load_library()
    mesh = lib_mod.Mesh(*periodic_kuhn_cube(7, "morton"))
    sizes = {}
    for elim in (1, 2):
        rc, h, _ = _create(mesh, k=2, elimination=elim)
        assert rc == 0
        ws, scratch, total = (ctypes.c_size_t() for _ in range(3))
        assert lib.dfdg_ctx_setup_bytes(h, ctypes.byref(ws), ctypes.byref(scratch)) == 0
        assert lib.dfdg_ctx_workspace_bytes(h, ctypes.byref(total)) == 0
        assert total.value == ws.value + scratch.value and ws.value % 256 == 0
        sizes[elim] = (ws.value, scratch.value)
        lib.dfdg_ctx_destroy(h)
    assert sizes[1][1] == 0 and sizes[2][0] < sizes[2][1]


@pytest.mark.gpu
def test_scratch_is_given_back():
    """Solves do not read the scratch after the bind (overwritten here), a bind with too little of
    it is refused, and one block for both parts gives the same solution."""
    from gpu_util import make_pair
    lib = lib_mod.load_library()
    _, s, _, _ = make_pair(20, 2, oracle=False, precond="amg", elimination=True)
    F = torch.randn(s.n_broken, generator=torch.Generator().manual_seed(2), dtype=torch.float64).to(s.device)
    U = s.mass_solve(F)[0]
    ws, scratch = ctypes.c_size_t(), ctypes.c_size_t()
    p, mesh = s.params, s.mesh
    out = []
    for split in (True, False):
        c = ctypes.c_void_p()
        assert lib.dfdg_ctx_create(mesh._h, ctypes.byref(p), ctypes.c_void_p(s.stream.cuda_stream), ctypes.byref(c)) == 0
        assert lib.dfdg_ctx_setup_bytes(c, ctypes.byref(ws), ctypes.byref(scratch)) == 0
        mem = torch.empty(ws.value + scratch.value + 512, dtype=torch.uint8, device=s.device)
        a = mem.data_ptr() + (-mem.data_ptr()) % 256
        if split:
            b = a + ws.value
            short = lib.dfdg_ctx_bind_workspace_scratch(c, ctypes.c_void_p(a), ws.value, ctypes.c_void_p(b), scratch.value - 1)
            assert short == -3 and lib.dfdg_ctx_bind_workspace_scratch(c, ctypes.c_void_p(a), ws.value, None, 0) == -3
            assert lib.dfdg_ctx_bind_workspace_scratch(c, ctypes.c_void_p(a), ws.value, ctypes.c_void_p(b), scratch.value) == 0
            mem[b - mem.data_ptr():].fill_(255)  # NaN
        else:
            assert lib.dfdg_ctx_bind_workspace(c, ctypes.c_void_p(a), ws.value + scratch.value - 1) == -3
            assert lib.dfdg_ctx_bind_workspace(c, ctypes.c_void_p(a), ws.value + scratch.value) == 0
        V = torch.empty_like(U)
        info = lib_mod.SolveInfo()
        assert lib.dfdg_hdiv_mass_solve(c, ctypes.c_void_p(F.data_ptr()), ctypes.c_void_p(V.data_ptr()), None,
                                        ctypes.byref(info)) == 0
        torch.cuda.synchronize()
        out.append(V)
        lib.dfdg_ctx_destroy(c)
    assert torch.equal(out[0], U) and torch.equal(out[1], U)
