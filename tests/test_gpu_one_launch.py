"""The one-launch solves of 2D systems on the GPU: every kernel variant (rows
a thread), one workgroup and many, ragged tiles, against the oracle's operator
(the residual of the solution, formed by the oracle in FP64) and its PCG's
iteration count; the fall back to one launch an iteration; two contexts at
once on two streams."""
import threading

import numpy as np
import pytest

from test_gpu_parity import FIELDS, cfg_mesh, compare, gea_mod, pair, rel  # noqa: F401

pytestmark = pytest.mark.gpu


def system(oracle_lib, gea_mod, name, nx, nz, solver, tol):  # noqa: F811
    cfg = cfg_mesh(name, nx, nz, tol=tol, max_iter=100000)
    O, s, S = pair(oracle_lib, gea_mod, cfg, solver=solver)
    print(f"[one launch] {nx}x{nz} {solver}", flush=True)
    S.step(1)  # the solve below starts from a state in motion
    x = np.ascontiguousarray(S.state()["pp"])
    st = S.pressure_solve(x)
    c, D, b = S.get_fields(gea_mod.FIELD_C | gea_mod.FIELD_D | gea_mod.FIELD_B)
    x0 = np.ascontiguousarray(S.state()["pp"])
    S.close()
    r = b - O.apply_A(c, D, x)
    return O, c, D, b, x0, x, st, float(np.linalg.norm(r) / np.linalg.norm(b))


# FP64: 2, 4, 8 and 16 rows a thread; one workgroup; partial tiles in x and z
@pytest.mark.parametrize("nx,nz", [(64, 32), (63, 31), (65, 33), (129, 20), (300, 70), (700, 450),
                                   (1000, 700), (1300, 900)])
def test_fp64_solve_matches_oracle(oracle_lib, gea_mod, nx, nz):  # noqa: F811
    tol = 1e-11
    O, c, D, b, x0, x, st, res = system(oracle_lib, gea_mod, "bubble2d_64x32" if nz < 100 else "paper_smooth_5m",
                                        nx, nz, "pcg64", tol)
    assert st.status == 0
    # (the solve stops on the recursive residual; the true one differs from
    # it by rounding, eps cond(A)^(1/2)-like, below a tenth of 1e-11)
    assert res <= 1.1 * tol
    if nx * nz <= 50000:
        xo, so, rc = O.pcg(c, D, b, x0, tol=tol)
        assert rc == 0 and abs(so.iters - st.iters) <= 1
        assert rel(x, xo) <= 1e-9


# FP32 inner solves: 2, 4, 8, 16 and 32 rows a thread
@pytest.mark.parametrize("nx,nz", [(60, 30), (257, 66), (700, 450), (1000, 700), (1500, 1000), (2048, 1100)])
def test_refined_solve_reaches_tolerance(oracle_lib, gea_mod, nx, nz):  # noqa: F811
    tol = 1e-9
    st, res = system(oracle_lib, gea_mod, "bubble2d_64x32" if nz < 100 else "paper_smooth_5m", nx, nz,
                     "mixed", tol)[6:]
    assert st.status == 0
    assert res <= 1.001 * tol  # (the refined forms stop on the true residual)


def test_given_up_solves_are_done_again(oracle_lib, gea_mod):  # noqa: F811
    cfg = cfg_mesh("bubble2d_64x32", 300, 70, tol=1e-13)
    O, s, S = pair(oracle_lib, gea_mod, cfg)
    assert S.L.gea_set_wait_limit(S.ctx, 0) == 0
    O.step(s, 2)
    st = S.step(2)
    assert st.steps_done == 2
    compare(S, s, 1e-10, cfg, 2)
    S.close()


def test_given_up_refined_solves_are_done_again(oracle_lib, gea_mod):  # noqa: F811
    # (the refined forms' bar: the residual they stop on; compare's floors are FP64's)
    cfg = cfg_mesh("bubble2d_64x32", 300, 70, tol=1e-9)
    O, s, S = pair(oracle_lib, gea_mod, cfg, solver="mixed")
    assert S.L.gea_set_wait_limit(S.ctx, 0) == 0
    x = s.pp.copy()
    st = S.pressure_solve(x)
    c, D, b = S.get_fields(gea_mod.FIELD_C | gea_mod.FIELD_D | gea_mod.FIELD_B)
    assert st.status == 0
    assert np.linalg.norm(b - O.apply_A(c, D, x)) <= 1.001e-9 * np.linalg.norm(b)
    assert S.step(2).steps_done == 2
    S.close()


def test_two_contexts_at_once(gea_mod):  # noqa: F811
    import torch
    cfg = cfg_mesh("paper_smooth_5m", 600, 400, tol=1e-10)
    ref = gea_mod.Solver(cfg["mesh"], cfg["params"], solver="pcg64")
    ref.init_bubble(**cfg["bubble"])
    ref.step(10)
    want = ref.state()
    ref.close()
    got = [None, None]

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            S = gea_mod.Solver(cfg["mesh"], cfg["params"], solver="pcg64")
            S.init_bubble(**cfg["bubble"])
            S.step(10)
            got[k] = S.state()
            S.close()

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for g in got:
        for f in FIELDS:
            assert np.array_equal(g[f], want[f]), f
