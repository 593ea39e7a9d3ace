"""max_iter of a refined solve caps the sum of its inner iterations, however
many inner solves went out before the host read one."""
import ctypes as C

import numpy as np
import pytest

from test_gpu_parity import cfg_mesh, gea_mod, pair  # noqa: F401

pytestmark = pytest.mark.gpu

MESHES = [("bubble2d_64x32", 64, 32, None), ("paper_smooth_5m", 300, 72, None), ("bubble3d_256x256x128", 40, 24, 20)]


# (below the first inner solve's iterations, among the later ones', short of the last)
@pytest.mark.parametrize("mesh", MESHES)
@pytest.mark.parametrize("solver", ["mixed", "learned"])
def test_pressure_solve_cap(oracle_lib, gea_mod, mesh, solver):  # noqa: F811
    name, nx, nz, ny = mesh
    tol = 1e-11
    cfg = cfg_mesh(name, nx, nz, ny, tol=tol, learned_always=1)
    O, s, S = pair(oracle_lib, gea_mod, cfg, solver=solver)
    if solver == "learned":
        S.load_weights()
    full = S.pressure_solve(s.pp.copy())
    assert full.outer_iters >= 2
    for cap in sorted({max(1, full.iters * k // 16) for k in range(1, 16)} | {full.iters - 1}):
        S.set_solver(solver, tol, max_iter=cap)
        x, st = s.pp.copy(), gea_mod.SolveStats()
        rc = S.L.gea_pressure_solve(S.ctx, None, C.c_void_p(x.ctypes.data), gea_mod.HOST, C.byref(st))
        print(f"[cap] {name} {nx}x{nz} {solver} cap {cap} of {full.iters}: {st.iters}, status {rc}", flush=True)
        assert st.iters <= cap
        assert rc == (gea_mod.OK if st.rel_res <= tol else gea_mod.ERR_NOCONV)
    S.close()


@pytest.mark.parametrize("mesh", MESHES)
@pytest.mark.parametrize("solver", ["mixed", "learned"])
def test_step_cap(oracle_lib, gea_mod, mesh, solver):  # noqa: F811
    # (after a step of its own a corrector's inner solves go out before their check is read)
    name, nx, nz, ny = mesh
    tol = 1e-11
    cfg = cfg_mesh(name, nx, nz, ny, tol=tol, learned_always=1)
    O, s, S = pair(oracle_lib, gea_mod, cfg, solver=solver)
    if solver == "learned":
        S.load_weights()
    full = S.step(2)
    most = max(full.solve[k].iters for k in range(full.n_solves))
    for cap in sorted({max(20, most * k // 8) for k in range(2, 8)}):
        S.set_solver(solver, tol, max_iter=cap)
        before = S.state()
        rc, st = S.step_status(1)
        iters = [st.solve[k].iters for k in range(st.n_solves)]
        print(f"[cap] {name} {nx}x{nz} {solver} step, cap {cap} of {most}: {iters}, status {rc}", flush=True)
        assert max(iters, default=0) <= cap
        if rc != gea_mod.OK:
            assert rc == gea_mod.ERR_NOCONV
            assert all(np.array_equal(before[f], v) for f, v in S.state().items())
    S.close()
