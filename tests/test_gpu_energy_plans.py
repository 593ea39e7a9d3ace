"""The energy sweeps' CG on 3D meshes whose fixed chunks leave CUs idle (the
iteration in short chunks, its sums in a pass of their own: one chunk, several,
uneven ones, tiles cut by the mesh) and on one where they do not, against the
oracle: the temperature of a step is their result alone."""
import numpy as np
import pytest

from test_gpu_parity import cfg_mesh, gea_mod, pair, rel  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(5, 4, 3), (64, 8, 64), (65, 9, 65), (130, 21, 37), (20, 12, 200), (250, 250, 70)])
@pytest.mark.parametrize("solver", ["mixed", "pcg64"])
def test_energy_sweeps_match_oracle(oracle_lib, gea_mod, dims, solver):  # noqa: F811
    nx, ny, nz = dims
    cfg = cfg_mesh("bubble3d_256x256x128", nx, nz, ny, tol=1e-9, max_iter=100000)
    # a diffusion number of 0.1: iterations enough, and Step 1's diffusion stable
    m, par = cfg["mesh"], cfg["params"]
    par["mu"] = 0.1 * min(m["lx"] / nx, m["ly"] / ny, m["lz"] / nz) ** 2 / par["dt"]
    O, s, S = pair(oracle_lib, gea_mod, cfg, solver=solver)
    print(f"[energy] {dims} {solver}", flush=True)
    # (temperatures that vary from cell to cell: the sweeps have work on every mesh)
    s.T += np.random.default_rng(3).uniform(-0.5, 0.5, s.T.shape)
    S.set_state(s.rho, np.ascontiguousarray(s.u), s.T, s.pp, s.p, s.Tbg)
    O.step(s, 1)
    st = S.step(1)
    assert st.energy_iters >= 2
    # (the sweeps are solved far below it; the parity bar of test_gpu_parity.py)
    assert rel(S.state()["T"], s.T) <= 1e-10
    S.close()
