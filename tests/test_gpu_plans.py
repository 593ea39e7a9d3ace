"""Launch plans of the marching kernels on the GPU: meshes whose chunks of
planes are cut to fill the card (one plane a chunk, uneven last chunks, more
than one full chunk) against the oracle, at the parity bar of
test_gpu_parity.py (1e-10 per field with both solves at 1e-13)."""
import pytest

from test_gpu_parity import cfg_mesh, compare, gea_mod, pair  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,dims", [
    ("bubble3d_256x256x128", (16, 16, 5)),     # one plane a chunk
    ("bubble3d_256x256x128", (130, 24, 37)),   # an uneven last chunk
    ("bubble3d_256x256x128", (24, 72, 67)),    # full chunks of 64 (and 32) cut in equal parts
    ("bubble2d_64x32", (65, 33, None)),        # one row a wave, waves of two rows in a workgroup
    ("bubble2d_64x32", (321, 129, None))])
def test_step_on_cut_chunks_matches_oracle(oracle_lib, gea_mod, name, dims):  # noqa: F811
    nx, nz, ny = (dims[0], dims[2], dims[1]) if dims[2] else (dims[0], dims[1], None)
    cfg = cfg_mesh(name, nx, nz, ny, tol=1e-13)
    O, s, S = pair(oracle_lib, gea_mod, cfg)
    print(f"[plans] {name} {nx}x{ny or 1}x{nz}", flush=True)
    O.step(s, 2)
    S.step(2)
    compare(S, s, 1e-10, cfg, 2)
    S.close()
