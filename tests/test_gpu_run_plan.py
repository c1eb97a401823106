"""The launches that lbm_run_plan lists are those the calls walk: their kernels, depths and
tiles, for default plans (regrouped) and for a depth asked for."""
import pytest

from gpu_helpers import W, gpu_solver, smooth_random_2d

pytestmark = pytest.mark.gpu

FACES = dict(bc=("inflow", "neumann", "wall", "inflow"), inflow={0: (1.1, 0.15, 0.05), 3: (1.0, 0.1, -0.1)})


def _steps(plan):
    return sum(l["steps"] for l in plan)


@pytest.mark.parametrize("nx,ny,kw,kernel", [
    (100, 60, {}, "tile"), (140, 80, FACES, "tile"), (300, 299, {}, "tile"), (633, 631, FACES, "tile"),
    (1024, 1024, {}, "strip"), (961, 1100, {}, "strip"), (1001, 1100, FACES, "strip")])
def test_default_2d_runs(nx, ny, kw, kernel):
    S = gpu_solver(smooth_random_2d(nx, ny, lam=6.0, s=1.7, **kw))
    for n in (0, 1, 2, 40, 72):
        plan = S.run_plan(n)
        assert _steps(plan) == n and all(l["steps"] >= 1 for l in plan)
        for l in plan:
            assert l["kernel"] == (kernel if l["steps"] > 1 else "step") or (n == 2 and l["kernel"] == "lds2")
            assert (l["rows"] > 0) == (l["steps"] > 1)
    most = max(l["steps"] for l in S.run_plan(72))
    assert len(S.run_plan(72)) == -(-72 // most)
    assert S.current()[1] == 0


@pytest.mark.parametrize("rest", [False, True])
def test_default_1d_runs(rest):
    from paper_1401_0427_amd.lbm import Solver
    import numpy as np

    for n, per in ((80, False), (80, True), (1000, False), (70000, True)):
        bc = ("periodic",) * 4 if per else ("neumann", "neumann", "periodic", "periodic")
        S = Solver(1, n, 1, lam=8.0, s=1.7, bc=bc, h0=np.ones(n), rest=rest, a=0.1 if rest else 0.0)
        plan = S.run_plan(400)
        assert _steps(plan) == 400 and all(l["kernel"] == "line" for l in plan)
        if n == 80 and not per:
            assert plan == [dict(kernel="line", steps=400, cols=80, rows=1)]
        elif not per:
            assert all(l["cols"] < n for l in plan)  # a tile holds one end at most


@pytest.mark.parametrize("n,fuse", [(200, 3), (1024, 5), (1024, 2)])
def test_a_depth_asked_for_is_kept(n, fuse):
    S = gpu_solver(smooth_random_2d(n, n), fuse_steps=fuse)
    for steps in (1, 7, 23):
        assert [l["steps"] for l in S.run_plan(steps)] == S.launch_plan(steps)


def test_state_checks_end_launches():
    S = gpu_solver(smooth_random_2d(100, 60), check_every=5)
    S.step(3)
    plan = S.run_plan(9)
    at = 3
    for l in plan:
        assert at // 5 == (at + l["steps"] - 1) // 5
        at += l["steps"]
    assert at == 12


@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_levels_and_adjoint_runs(storage):
    for nx, ny, levels, sweep in ((96, 64, "tile", "tile"), (512, 512, "tile", "strip"), (1024, 1024, "strip", "strip")):
        S = gpu_solver(smooth_random_2d(nx, ny), storage=storage)
        for n in (1, 2, 9, 24):
            L, A = S.run_plan(n, "levels"), S.run_plan(n, "adjoint")
            assert _steps(L) == n and _steps(A) == n
            assert len(A) % 2 == n % 2  # lambda ends in the buffer that single steps end in
        assert L[0]["kernel"] == levels and A[0]["kernel"] == sweep
    S = gpu_solver(smooth_random_2d(96, 64, **FACES), storage=storage)
    assert all(l["kernel"] == "step" for l in S.run_plan(9, "adjoint"))
    S = gpu_solver(W.dam_break_1d(100), storage=storage)
    assert all(l["kernel"] == "step" for r in ("levels", "adjoint") for l in S.run_plan(9, r))


def test_rejected():
    from paper_1401_0427_amd import lbm

    S = gpu_solver(smooth_random_2d(20, 20))
    L = lbm.load()
    assert L.lbm_run_plan(S.ctx, 3, 5, None, 0, None) == lbm.LBM_EINVAL
    assert L.lbm_run_plan(S.ctx, 0, -1, None, 0, None) == lbm.LBM_EINVAL
    assert L.lbm_run_plan(S.ctx, 0, 5, None, 2, None) == lbm.LBM_EINVAL
    R = gpu_solver(smooth_random_2d(20, 20), rest=True, a=0.05)
    assert L.lbm_run_plan(R.ctx, 2, 5, None, 0, None) == lbm.LBM_EINVAL
    assert L.lbm_run_plan(None, 0, 5, None, 0, None) == lbm.LBM_ESTATE


@pytest.mark.parametrize("n,rest,faces,steps,lone", [
    (2048, False, False, 10, True), (2048, False, False, 19, False), (2048, False, False, 100, False),
    (1500, False, False, 10, False), (2048, False, True, 50, True), (3000, False, True, 22, True),
    (3000, False, True, 78, False), (2048, True, False, 67, True), (3000, True, False, 67, False)])
def test_one_step_left_over(n, rest, faces, steps, lone):
    """A remainder of one step is a launch of its own only where the deeper launches that
    it leaves cost less than spreading it."""
    import torch

    from paper_1401_0427_amd.lbm import Solver

    kw = dict(rest=True, a=0.05, rates=[1.7] * 10) if rest else {}
    S = Solver(2, n, n, lam=6.0, s=1.7, h0=torch.ones(n, n, dtype=torch.float64).numpy(),
               **(FACES if faces else {}), **kw)
    depths = [l["steps"] for l in S.run_plan(steps)]
    most = max(depths)
    assert sum(depths) == steps and len(depths) == -(-steps // max(most, 6))
    assert (depths[-1] == 1 and set(depths[:-1]) == {most}) == lone
    if not lone:
        assert most - min(depths) <= 1
