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
