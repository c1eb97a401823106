"""Wave-strip launches of default plans (their own depth and segments): bit for bit equal
to single steps, at every depth a run can take, on grids just beyond the tile launches."""
import pytest

from gpu_helpers import gpu_solver, smooth_random_2d

pytestmark = pytest.mark.gpu

FACES = ("inflow", "neumann", "wall", "inflow")


@pytest.mark.parametrize("storage,faces,nx,ny", [
    ("f64", False, 1024, 1024), ("f64", False, 961, 1100), ("f64", False, 5000, 330),
    ("f64", True, 1001, 1100), ("f64", True, 90, 14000), ("f32", False, 1501, 1333),
    ("f32", True, 1480, 1501), ("f64", False, 610, 607), ("f32", False, 730, 701),
    ("f64", True, 901, 870), ("f32", True, 1350, 1340)])
def test_default_strips_equal_single_steps(storage, faces, nx, ny):
    """Ragged last strips and segments, few and many segments to a column; runs that take
    one launch of 2 .. 9 steps each, and one that takes several."""
    import torch

    kw = dict(bc=FACES, inflow={0: (1.1, 0.15, 0.05), 3: (1.0, 0.1, -0.1)}) if faces else {}
    case = smooth_random_2d(nx, ny, seed=nx % 5, lam=6.0, s=1.7, **kw)
    A = gpu_solver(case, storage=storage, fuse_steps=1)
    B = gpu_solver(case, storage=storage)
    for n in (2, 3, 4, 5, 6, 7, 8, 9, 21):
        A.step(n)
        B.step(n)
        assert torch.equal(A.planes(), B.planes()), n


RATES = [1.7, 1.6, 1.5, 1.4, 1.8, 1.75, 1.3, 1.65, 1.85, 1.2]


@pytest.mark.parametrize("storage,fuse,nx,ny,runs", [
    ("f64", 0, 561, 530, (2, 3, 4, 5, 13)), ("f64", 0, 1024, 1024, (5, 12)),
    ("f32", 0, 763, 751, (2, 3, 4, 5, 6, 7, 15)), ("f64", 0, 300, 2000, (5, 8)),
    ("f64", 5, 4600, 4599, (5, 7)), ("f32", 4, 6500, 6401, (4, 3))])
def test_rest_population_strips_equal_single_steps(storage, fuse, nx, ny, runs):
    """D2Q5Q4Q4 strips of default plans at every depth, and grids whose planes together
    reach 2 GiB (a buffer descriptor per plane)."""
    import torch

    from paper_1401_0427_amd.lbm import Solver

    c = smooth_random_2d(nx, ny, seed=3, lam=6.0, s=1.7)
    A, B = (Solver(2, nx, ny, lam=c.lam, s=c.s, h0=c.h0, qx0=c.qx0, qy0=c.qy0, storage=storage,
                   rest=True, a=0.05, rates=RATES, fuse_steps=f) for f in (1, fuse))
    for n in runs:
        A.step(n)
        B.step(n)
        assert torch.equal(A.planes(), B.planes()), n
