"""Adjoint sweeps and stored levels of flat, narrow and long grids: the launches they take,
bit for bit those of single steps."""
import pytest

from gpu_helpers import gpu_solver, smooth_random_2d
from test_gpu_adjoint_multi import test_sweeps_equal_single_steps as sweeps_equal_single_steps

pytestmark = pytest.mark.gpu

FACES = dict(bc=("inflow", "neumann", "wall", "inflow"), inflow={0: (1.1, 0.15, 0.05), 3: (1.0, 0.1, -0.1)})


@pytest.mark.parametrize("storage,adj", [("f64", None), ("f32", "f32"), ("f32", "f64")])
@pytest.mark.parametrize("nx,ny", [(1001, 2), (6144, 8), (6145, 8), (20000, 3), (37501, 2), (200, 225), (128, 512),
                                   (8, 1501), (9, 1501), (3, 20001), (385, 384), (2000, 61)])
def test_sweeps(nx, ny, storage, adj):
    """Both sides of every limit: tiles of each shape just running at once or not, the sizes
    from which strips take two steps, narrow grids in one column of tiles."""
    sweeps_equal_single_steps(nx, ny, storage, adj)


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny,kw", [(100001, 3, FACES), (30001, 8, FACES), (8, 3001, FACES), (401, 400, FACES),
                                      (949, 948, FACES), (40001, 9, {}), (64, 4097, {}), (90001, 16, {}),
                                      (90001, 17, {})])
def test_levels(nx, ny, kw, storage):
    import torch

    S = gpu_solver(smooth_random_2d(nx, ny, seed=2, **kw), storage=storage)
    nb = S.nplanes * S.ps
    prev = S.current()[0].clone()
    levels = S.new_state(7)
    S.step_levels(prev, 7, levels)
    for i in range(7):
        nxt = S.new_state()
        S.step_buffers(prev, nxt)
        assert torch.equal(S.planes(nxt), S.planes(levels[i * nb:(i + 1) * nb])), (i, S.run_plan(7, "levels"))
        prev = nxt


@pytest.mark.parametrize("nx,ny,kw,storage,run,kernel,cols", [
    (300000, 2, FACES, "f64", "levels", "step", 0),   # in tiles 8 times as long
    (100000, 3, FACES, "f32", "levels", "step", 0),   # 2.2
    (400, 400, FACES, "f64", "levels", "tile", 32),   # 64 x 32 tiles spill: 1.8
    (700, 700, FACES, "f64", "levels", "tile", 32),   # 1.6
    (1000000, 3, {}, "f32", "levels", "step", 0),     # in strips 1.3
    (20000, 3, {}, "f64", "adjoint", "step", 0),      # in tiles 1.3
    (4096, 16, {}, "f64", "adjoint", "tile", 32)])    # in tiles of 32 x 16 1.15
def test_no_launch_that_is_slower_than_single_steps(nx, ny, kw, storage, run, kernel, cols):
    S = gpu_solver(smooth_random_2d(nx, ny, **kw), storage=storage)
    plan = S.run_plan(20, run)
    assert all(l["kernel"] == kernel and l["cols"] == cols for l in plan if l["steps"] > 1 or kernel == "step")
