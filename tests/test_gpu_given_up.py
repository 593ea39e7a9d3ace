"""One-launch solves that are given up (a workgroup's wait outlasts the limit,
here 0: at its first poll): the call is done again with one launch an
iteration, which the launch counts show, and its result is the solve's."""
import numpy as np
import pytest

from test_gpu_parity import cfg_mesh, gea_mod, pair  # noqa: F401

pytestmark = pytest.mark.gpu


def context(oracle_lib, gea_mod, dims, solver, **par):  # noqa: F811
    nx, ny, nz = dims
    name = "bubble3d_256x256x128" if ny else "bubble2d_64x32"
    cfg = cfg_mesh(name, nx, nz, ny or None, **par)
    print(f"[given up] {dims} {solver}", flush=True)
    return (*pair(oracle_lib, gea_mod, cfg, solver=solver), cfg)


# every form of the exchange: A p in 2D and 3D, the direction in 3D, vectors on
# the chip and in memory; many workgroups of which some end well
@pytest.mark.parametrize("dims,solver", [((300, 0, 70), "pcg64"), ((1000, 0, 700), "pcg64"), ((700, 0, 450), "mixed"),
                                         ((90, 60, 40), "pcg64"), ((128, 128, 100), "pcg64"),
                                         ((150, 90, 61), "mixed"), ((250, 110, 250), "mixed")])
def test_a_given_up_solve_is_done_again(oracle_lib, gea_mod, dims, solver):  # noqa: F811
    tol = 1e-11 if solver == "pcg64" else 1e-9
    O, s, S, cfg = context(oracle_lib, gea_mod, dims, solver, tol=tol, max_iter=100000)
    assert S.L.gea_set_wait_limit(S.ctx, 0) == 0
    S.kernel_timing(True)
    x = s.pp.copy()
    st = S.pressure_solve(x)
    launches = S.kernel_times()[1][0 if solver == "pcg64" else 2]
    S.kernel_timing(False)
    c, D, b = S.get_fields(gea_mod.FIELD_C | gea_mod.FIELD_D | gea_mod.FIELD_B)
    S.close()
    assert st.status == 0 and st.iters > 0
    assert launches > st.iters  # (one an iteration, and the given-up solve)
    # (the recursive residual of the FP64 form is within a tenth of 1e-11 of the true one)
    assert np.linalg.norm(b - O.apply_A(c, D, x)) <= (1.1 if solver == "pcg64" else 1.001) * tol * np.linalg.norm(b)


# A solve given up in a step that ends with another solve's error: behind it (a
# single workgroup's refined pressure solve behind a given-up energy sweep), or
# before it (an energy sweep short of iterations before a given-up pressure
# solve).  The step is rolled back, and what the given-up launch left in the
# exchange area is not taken for a later solve's.
@pytest.mark.parametrize("dims,solver,max_iter", [((64, 0, 32), "mixed", 3), ((200, 0, 16), "pcg64", 1)])
def test_given_up_beside_another_error(oracle_lib, gea_mod, dims, solver, max_iter):  # noqa: F811
    tol = 1e-11 if solver == "pcg64" else 1e-9
    O, s, S, cfg = context(oracle_lib, gea_mod, dims, solver, tol=tol, max_iter=max_iter)
    before = S.state()
    assert S.L.gea_set_wait_limit(S.ctx, 0) == 0
    for _ in range(2):
        assert S.step_status(1)[0] == gea_mod.ERR_NOCONV
        for f, v in S.state().items():
            assert np.array_equal(before[f], v), f
    assert S.L.gea_set_wait_limit(S.ctx, 25000000) == 0
    S.set_solver(solver, tol, max_iter=100000)
    assert S.step(3).steps_done == 3
    x = np.ascontiguousarray(S.state()["pp"])
    assert S.pressure_solve(x).status == 0
    c, D, b = S.get_fields(gea_mod.FIELD_C | gea_mod.FIELD_D | gea_mod.FIELD_B)
    S.close()
    assert np.linalg.norm(b - O.apply_A(c, D, x)) <= (1.1 if solver == "pcg64" else 1.001) * tol * np.linalg.norm(b)


# A launch that needs most of the card beside small ones on other streams, each
# partly placed, would wait for each other: their shares keep them apart (no
# solve takes one launch an iteration), and nothing else changes.
def test_large_and_small_solves_at_once(gea_mod):  # noqa: F811
    import threading

    import torch
    jobs = [((600, 400), 12), ((300, 70), 40), ((200, 120), 40)]  # about 250, 25 and 32 workgroups
    cfgs = [cfg_mesh("paper_smooth_5m", nx, nz, tol=1e-10) for (nx, nz), _ in jobs]

    def run(k):
        S = gea_mod.Solver(cfgs[k]["mesh"], cfgs[k]["params"], solver="pcg64")
        S.init_bubble(**cfgs[k]["bubble"])
        S.kernel_timing(True)
        st = S.step(jobs[k][1])
        launches = S.kernel_times()[1]
        S.kernel_timing(False)
        out = S.state()
        S.close()
        return st, launches, out

    alone = [run(k) for k in range(3)]
    got = [None] * 3

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            got[k] = run(k)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for (st, launches, out), (_, _, want) in zip(got, alone):
        assert launches[0] == st.total_solves  # (pressure solves; class 7: a set-up and a solve a sweep)
        assert launches[7] == 4 * st.steps_done
        for f, v in want.items():
            assert np.array_equal(out[f], v), f


# One give-up is not for good: the steps after it pause, twice as long after the
# next, and then take one launch a solve again; the count tells.
@pytest.mark.parametrize("dims", [(64, 0, 32), (300, 0, 70), (40, 24, 20)])
def test_one_launch_solves_come_back(oracle_lib, gea_mod, dims):  # noqa: F811
    S = context(oracle_lib, gea_mod, dims, "pcg64", tol=1e-11)[2]

    def one_launch_a_solve(steps):  # (a step of two pressure solves takes more than two iterations)
        S.kernel_timing(True)
        st = S.step(steps)
        n = S.kernel_times()[1][0]
        S.kernel_timing(False)
        assert n == st.total_solves or n >= st.total_iters > st.total_solves
        return n == st.total_solves

    assert one_launch_a_solve(2) and S.given_up() == 0
    for pause in (64, 128):
        assert S.L.gea_set_wait_limit(S.ctx, 0) == 0
        assert not one_launch_a_solve(1)  # (tried, done again: the first of the pause)
        assert S.L.gea_set_wait_limit(S.ctx, 25000000) == 0
        n = S.given_up()
        assert n == (1 if pause == 64 else 2)
        assert not one_launch_a_solve(1)
        S.step(pause - 4)
        assert not one_launch_a_solve(1)  # (the last of it: step number pause - 1, the try being one)
        assert one_launch_a_solve(2) and S.given_up() == n
    S.close()


# The static solve: done again from the initial guess (workgroups that ended well
# beside the one that gave up have written their part of x), with nothing left
# for the next call.
@pytest.mark.parametrize("dims", [(333, 0, 251), (60, 50, 40)])
def test_a_given_up_static_solve_is_done_again(oracle_lib, gea_mod, dims):  # noqa: F811
    import ctypes as C

    import torch
    tol = 1e-11
    O, s, S, cfg = context(oracle_lib, gea_mod, dims, "pcg64", tol=1e-9)
    S.step(1)
    x0 = S.state()["pp"]
    S.pressure_solve(np.ascontiguousarray(x0))
    c, D, b = S.get_fields(gea_mod.FIELD_C | gea_mod.FIELD_D | gea_mod.FIELD_B)
    mesh, L = S.mesh, S.L
    S.close()
    dev = [torch.tensor(v, device="cuda:0") for v in (c, D, b)]

    def solve(ticks):
        x, st, n = torch.tensor(x0, device="cuda:0"), gea_mod.SolveStats(), C.c_int32(-1)
        rc = L.gea_pressure_solve_static_wait(C.byref(mesh), *[C.c_void_p(t.data_ptr()) for t in (*dev, x)], tol, 20000,
                                              C.c_void_p(torch.cuda.current_stream().cuda_stream), ticks, C.byref(n),
                                              C.byref(st))
        assert rc == gea_mod.OK
        x = x.cpu().numpy()
        assert np.linalg.norm(b - O.apply_A(c, D, x)) <= 1.1 * tol * np.linalg.norm(b)
        return x, st, n.value

    x1, st1, n1 = solve(25000000)
    assert n1 == 0
    x2, st2, n2 = solve(0)
    assert n2 == 1 and st2.rel_res0 == st1.rel_res0 and abs(st2.iters - st1.iters) <= 1
    for _ in range(4):
        x, st, n = solve(0)
        assert n == 1 and st.iters == st2.iters and np.array_equal(x, x2)
    x, st, n = solve(25000000)
    assert n == 0 and st.iters == st1.iters and np.array_equal(x, x1)


# A static mesh whose exchange does not fit the static area (96 x 96 x 48: 144
# tiles of 64 x 8 x 8) takes the iteration kernels.
def test_static_mesh_above_the_exchange_area(gea_mod):  # noqa: F811
    import ctypes as C

    import torch
    mesh = gea_mod.make_mesh(dict(nx=96, ny=96, nz=48, lx=960.0, ly=960.0, lz=480.0))
    n = 96 * 96 * 48
    b = torch.rand(n, generator=torch.Generator().manual_seed(3), dtype=torch.float64).cuda()
    c, D, x = torch.full_like(b, 0.01), torch.full_like(b, 0.01), torch.zeros_like(b)
    st, up = gea_mod.SolveStats(), C.c_int32(-1)
    rc = gea_mod.lib().gea_pressure_solve_static_wait(
        C.byref(mesh), *[C.c_void_p(t.data_ptr()) for t in (c, D, b, x)], 1e-10, 20000,
        C.c_void_p(torch.cuda.current_stream().cuda_stream), 0, C.byref(up), C.byref(st))
    assert rc == gea_mod.OK and st.rel_res <= 1e-10 and st.iters > 1
    assert up.value == 0  # (no one-launch solve that could give up)
    # the residual with a uniform D: c x + D (S/h) (differences to the neighbours)
    v = x.view(48, 96, 96)
    r = b.view(48, 96, 96) - 0.01 * v
    for d in range(3):
        f = 0.01 * 10.0 * (v.narrow(d, 1, v.shape[d] - 1) - v.narrow(d, 0, v.shape[d] - 1))
        r.narrow(d, 0, v.shape[d] - 1).add_(f)
        r.narrow(d, 1, v.shape[d] - 1).sub_(f)
    assert float(r.norm() / b.norm()) <= 1.1e-10
