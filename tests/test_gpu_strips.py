"""Wave-strip launches of default plans (their own depth and segments): bit for bit equal
to single steps, at every depth a run can take, on grids just beyond the tile launches."""
import pytest

from gpu_helpers import gpu_solver, smooth_random_2d

pytestmark = pytest.mark.gpu

FACES = ("inflow", "neumann", "wall", "inflow")


@pytest.mark.parametrize("storage,faces,nx,ny", [
    ("f64", False, 1024, 1024), ("f64", False, 961, 1100), ("f64", False, 5000, 330),
    ("f64", True, 1001, 1100), ("f64", True, 90, 14000), ("f32", False, 1501, 1333),
    ("f32", True, 1480, 1501)])
def test_default_strips_equal_single_steps(storage, faces, nx, ny):
    """Ragged last strips and segments, few and many segments to a column; runs that take
    one launch of 2 .. 9 steps each, and one that takes several."""
    import torch

    kw = dict(bc=FACES, inflow={0: (1.1, 0.15, 0.05), 3: (1.0, 0.1, -0.1)}) if faces else {}
    case = smooth_random_2d(nx, ny, seed=nx % 5, lam=6.0, s=1.7, **kw)
    A = gpu_solver(case, storage=storage, fuse_steps=1)
    B = gpu_solver(case, storage=storage)
    assert B.launch_info()["steps_per_launch"] >= 6
    for n in (2, 3, 4, 5, 6, 7, 8, 9, 21):
        A.step(n)
        B.step(n)
        assert torch.equal(A.planes(), B.planes()), n
