"""The one-launch solves of 3D systems on the GPU: every kernel variant (cells
a thread, vectors in registers or in memory, either exchange), one workgroup
and many, tiles cut by the mesh in each direction, against the oracle's
operator and its PCG's iteration count; the fall back to one launch an
iteration; steps on meshes of several tiles."""
import numpy as np
import pytest

from test_gpu_parity import gea_mod  # noqa: F401
from test_gpu_parity import cfg_mesh, compare, pair, rel

pytestmark = pytest.mark.gpu

NAME = "bubble3d_256x256x128"


def system3(oracle_lib, gea_mod, dims, solver, tol):  # noqa: F811
    nx, ny, nz = dims
    cfg = cfg_mesh(NAME, nx, nz, ny, tol=tol, max_iter=100000)
    O, s, S = pair(oracle_lib, gea_mod, cfg, solver=solver)
    print(f"[one launch] {nx}x{ny}x{nz} {solver}", flush=True)
    S.step(1)  # the solve below starts from a state in motion
    x = np.ascontiguousarray(S.state()["pp"])
    st = S.pressure_solve(x)
    c, D, b = S.get_fields(gea_mod.FIELD_C | gea_mod.FIELD_D | gea_mod.FIELD_B)
    x0 = np.ascontiguousarray(S.state()["pp"])
    S.close()
    r = b - O.apply_A(c, D, x)
    return O, c, D, b, x0, x, st, float(np.linalg.norm(r) / np.linalg.norm(b))


# FP64: 2, 4, 8 and 16 cells a thread
@pytest.mark.parametrize("dims", [(64, 8, 2), (65, 9, 3), (30, 20, 12), (90, 60, 40), (130, 70, 61), (128, 128, 100)])
def test_fp64_solve_matches_oracle(oracle_lib, gea_mod, dims):  # noqa: F811
    tol = 1e-11
    O, c, D, b, x0, x, st, res = system3(oracle_lib, gea_mod, dims, "pcg64", tol)
    assert st.status == 0
    # (the solve stops on the recursive residual; the true one differs from
    # it by rounding, eps cond(A)^(1/2)-like, below a tenth of 1e-11)
    assert res <= 1.1 * tol
    if np.prod(dims) <= 50000:
        xo, so, rc = O.pcg(c, D, b, x0, tol=tol)
        assert rc == 0 and abs(so.iters - st.iters) <= 1
        assert rel(x, xo) <= 1e-9


# FP32 inner solves: 2, 4, 16, 32 and 64 cells a thread (the last with x, c and
# D in memory)
@pytest.mark.parametrize("dims", [(60, 30, 9), (150, 90, 40), (150, 90, 61), (190, 120, 100), (250, 250, 110)])
def test_refined_solve_reaches_tolerance(oracle_lib, gea_mod, dims):  # noqa: F811
    tol = 1e-9
    st, res = system3(oracle_lib, gea_mod, dims, "mixed", tol)[6:]
    assert st.status == 0
    assert res <= 1.001 * tol  # (the refined forms stop on the true residual)


@pytest.mark.parametrize("limit", [None, 0])
def test_steps_match_oracle(oracle_lib, gea_mod, limit):  # noqa: F811
    # (limit 0: every launch of more than one workgroup gives up, and the
    # step is done again with the iteration kernels)
    cfg = cfg_mesh(NAME, 70, 21, 37, tol=1e-13)
    O, s, S = pair(oracle_lib, gea_mod, cfg)
    if limit is not None:
        assert S.L.gea_set_wait_limit(S.ctx, limit) == 0
    O.step(s, 2)
    assert S.step(2).steps_done == 2
    compare(S, s, 1e-10, cfg, 2)
    S.close()


def test_given_up_refined_solve_is_done_again(oracle_lib, gea_mod):  # noqa: F811
    # x is updated in memory by the variant of this mesh: the second solve has
    # to start where the first did
    cfg = cfg_mesh(NAME, 250, 110, 250, tol=1e-9)
    O, s, S = pair(oracle_lib, gea_mod, cfg, solver="mixed")
    assert S.L.gea_set_wait_limit(S.ctx, 0) == 0
    x = s.pp.copy()
    st = S.pressure_solve(x)
    c, D, b = S.get_fields(gea_mod.FIELD_C | gea_mod.FIELD_D | gea_mod.FIELD_B)
    assert st.status == 0
    assert np.linalg.norm(b - O.apply_A(c, D, x)) <= 1.001e-9 * np.linalg.norm(b)
    S.close()
