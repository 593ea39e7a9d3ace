"""Steps whose one-launch solves are read with the step's last read: what they
report is what solves read one by one report, and a solve that does not end
well leaves the state and the error as before."""
import numpy as np
import pytest

from test_gpu_parity import FIELDS, cfg_mesh, gea_mod, pair  # noqa: F401

pytestmark = pytest.mark.gpu

MESHES = [("bubble2d_64x32", 64, 32, None), ("paper_smooth_5m", 300, 70, None), ("bubble3d_256x256x128", 40, 24, 20)]


@pytest.mark.parametrize("mesh", MESHES)
def test_statistics_match_solves_read_one_by_one(oracle_lib, gea_mod, mesh):  # noqa: F811
    name, nx, nz, ny = mesh
    cfg = cfg_mesh(name, nx, nz, ny, tol=1e-11)
    O, s, A = pair(oracle_lib, gea_mod, cfg)
    B = pair(oracle_lib, gea_mod, cfg)[2]
    assert B.L.gea_set_wait_limit(B.ctx, 0) == 0  # (B: one launch an iteration, a read a solve)
    a, b = A.step(3), B.step(3)
    assert a.steps_done == b.steps_done == 3 and a.n_solves == b.n_solves and a.total_solves == b.total_solves
    # (iteration counts may differ by one a solve where the sums' order decides)
    assert abs(a.total_iters - b.total_iters) <= a.total_solves
    assert abs(a.energy_iters - b.energy_iters) <= 6
    for k in range(a.n_solves):
        assert a.solve[k].status == 0 and 0 < a.solve[k].rel_res <= 1e-11
        assert abs(a.solve[k].rel_res0 - b.solve[k].rel_res0) <= 1e-6 * b.solve[k].rel_res0
    A.close()
    B.close()


@pytest.mark.parametrize("mesh", MESHES)
def test_a_solve_that_does_not_converge_rolls_back(oracle_lib, gea_mod, mesh):  # noqa: F811
    name, nx, nz, ny = mesh
    cfg = cfg_mesh(name, nx, nz, ny, tol=1e-13, max_iter=3)
    O, s, S = pair(oracle_lib, gea_mod, cfg)
    before = S.state()
    for _ in range(2):  # (the second with a read behind each solve)
        with pytest.raises(gea_mod.GeaError) as err:
            S.step(1)
        assert "did not converge" in str(err.value)
        after = S.state()
        for f in FIELDS:
            assert np.array_equal(before[f], after[f]), f
    S.close()
