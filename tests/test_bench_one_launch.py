"""bench.py names the CG kernel that ran: the iteration kernel, or, where no
scalar kernel went out behind one, the one-launch solve, with the bytes that
one has to move."""
import pytest

from test_bench_host import load_bench

BIG = dict(nx=256, ny=256, nz=128)     # 512 tiles of 64 x 16 x 16: x, c and D in memory
SMALL = dict(nx=150, ny=90, nz=61)     # 72 tiles
PLANE = dict(nx=2048, ny=1, nz=2048)


@pytest.mark.parametrize("mesh,it_class,name,per_cell", [
    (BIG, 2, "k_cgp3<fp32>", 16 + 28 * 2 / 12), (SMALL, 2, "k_cgp3<fp32>", 36 * 2 / 12),
    (SMALL, 0, "k_cgp3<fp64>", 48 * 2 / 12), (PLANE, 2, "k_cgp2<fp32>", 36 * 2 / 12)])
def test_a_one_launch_solve_is_named(mesh, it_class, name, per_cell):
    b = load_bench()
    kms, kn = [0.0] * 8, [0] * 8
    kms[it_class], kn[it_class] = 3.0, 9
    got, c = b.cg_candidate(mesh, it_class, kms, kn, [9.9] * 4, 12.0, 2, 3)
    nc = mesh["nx"] * mesh["ny"] * mesh["nz"]
    assert got == name and abs(c["bytes_alg"] - per_cell * nc) < 1e-6 * nc
    assert abs(c["per_step_ms"] - 1.0) < 1e-12 and abs(c["avg_ms"] - 1.0 / 12) < 1e-12
    e = b.roofline_entry(dict(kernel=got, **c))
    assert "iteration" in e["per"] and abs(e["achieved"] - per_cell * nc * 12 / 1e6) < 0.1


def test_iteration_kernels_are_named():
    b = load_bench()
    kms, kn = [0.0] * 8, [0] * 8
    kms[2], kn[2], kn[3] = 3.0, 30, 4
    got, c = b.cg_candidate(BIG, 2, kms, kn, [0.1, 0.01, 0.08, 0.01], 10.0, 2, 3)
    assert got == "k_cg_iter<fp32>" and abs(c["per_step_ms"] - 0.8) < 1e-12
    assert "per" not in b.roofline_entry(dict(kernel=got, **c))
