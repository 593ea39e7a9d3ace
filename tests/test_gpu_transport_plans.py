"""The implicit transport solves of the refined form on 3D meshes whose fixed
chunks leave CUs idle (operator kernels in short chunks, sums in a pass of
their own) and on those where they do not, against the oracle: the
temperature of a step is their result alone."""
import pytest

from test_gpu_parity import cfg_mesh, gea_mod, pair, rel  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("dims", [(16, 12, 4), (70, 21, 37), (64, 9, 67), (33, 8, 130)])
def test_transport_of_the_refined_form_matches_oracle(oracle_lib, gea_mod, dims, form):  # noqa: F811
    nx, ny, nz = dims
    cfg = cfg_mesh("bubble3d_256x256x128", nx, nz, ny, tol=1e-9, max_iter=100000, energy_form=form, transport=1)
    O, s, S = pair(oracle_lib, gea_mod, cfg, solver="mixed")
    print(f"[transport] {dims} form {form}", flush=True)
    O.step(s, 1)
    st = S.step(1)
    assert st.transport_iters >= 1 + O.ndim
    # (both solves stop at 1e-13; the parity bar of test_gpu_parity.py)
    assert rel(S.state()["T"], s.T) <= 1e-10
    S.close()
