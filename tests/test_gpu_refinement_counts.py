"""outer_iters counts the refinement steps that were left to do: none where the
initial guess passes the residual check, also when an inner solve went out
behind that check before the host read it."""
import numpy as np
import pytest

from test_gpu_parity import cfg_mesh, gea_mod, pair  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mesh", [("bubble2d_64x32", 64, 32, None), ("paper_smooth_5m", 300, 72, None),
                                  ("bubble3d_256x256x128", 40, 24, 20)])
@pytest.mark.parametrize("solver", ["mixed", "learned"])
def test_outer_iterations_are_those_that_iterated(oracle_lib, gea_mod, mesh, solver):  # noqa: F811
    name, nx, nz, ny = mesh
    cfg = cfg_mesh(name, nx, nz, ny, tol=1e-8, learned_always=1)
    O, s, S = pair(oracle_lib, gea_mod, cfg, solver=solver)
    if solver == "learned":
        S.load_weights()
    for _ in range(3):  # (the first step predicts nothing of its checks)
        st = S.step(1)
        for k in range(st.n_solves):
            assert (st.solve[k].iters > 0) == (st.solve[k].outer_iters > 0), (k, st.solve[k].as_dict())
    x = np.ascontiguousarray(S.state()["pp"])
    first, again = S.pressure_solve(x), S.pressure_solve(x)
    assert first.iters > 0 and first.outer_iters > 0
    assert again.iters == 0 and again.outer_iters == 0 and again.status == 0
    S.close()


# b = 0: x = 0 without an iteration, from any guess (an inner solve that went
# out before the check's ||b|| was read does not count)
@pytest.mark.parametrize("mesh", [("bubble2d_64x32", 64, 32, None), ("paper_smooth_5m", 300, 72, None),
                                  ("bubble3d_256x256x128", 40, 24, 20)])
@pytest.mark.parametrize("solver", ["pcg64", "mixed", "learned"])
@pytest.mark.parametrize("guess", [0.0, 1.0, 1e60])
def test_no_right_hand_side(oracle_lib, gea_mod, mesh, solver, guess):  # noqa: F811
    name, nx, nz, ny = mesh
    cfg = cfg_mesh(name, nx, nz, ny, tol=1e-8)
    O, s, S = pair(oracle_lib, gea_mod, cfg, solver=solver)
    if solver == "learned":
        S.load_weights()
    S.step(1)
    x = np.full(S.nc, guess)
    st = S.pressure_solve(x, b=np.zeros(S.nc))
    S.close()
    assert not x.any()
    assert (st.status, st.iters, st.outer_iters, st.rel_res) == (0, 0, 0, 0.0)
