"""Default runs of grids a few rows high or a few columns wide: which launches they take,
and every one bit for bit equal to single steps."""
import pytest

from gpu_helpers import smooth_random_2d

pytestmark = pytest.mark.gpu

RATES = [1.7, 1.6, 1.5, 1.4, 1.8, 1.75, 1.3, 1.65, 1.85, 1.2]
FACES = ("inflow", "neumann", "wall", "inflow")


def _solver(nx, ny, faces, rest, storage, fuse):
    from paper_1401_0427_amd.lbm import Solver

    c = smooth_random_2d(nx, ny, seed=nx + ny, lam=6.0, s=1.7)
    return Solver(2, nx, ny, lam=c.lam, s=c.s, bc=FACES if faces else ("periodic",) * 4,
                  inflow={0: (1.1, 0.15, 0.05), 3: (1.0, 0.1, -0.1)} if faces else {}, h0=c.h0, qx0=c.qx0,
                  qy0=c.qy0, storage=storage, rest=rest, a=0.05 if rest else 0.0,
                  rates=RATES if rest else None, fuse_steps=fuse)


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("rest", [False, True])
@pytest.mark.parametrize("faces", [False, True])
def test_short_grids_equal_single_steps(faces, rest, storage):
    """Both sides of every limit of the rule: rows at which the depth of strips changes,
    sizes from a few tiles to many times the resident ones."""
    import torch

    for nx, ny in ((2501, 2), (20480, 4), (20481, 4), (9000, 9), (30001, 2), (60000, 3), (40001, 8),
                   (200000, 2), (250001, 4), (2, 2600), (3, 30001), (8, 5001), (9, 5001)):
        A = _solver(nx, ny, faces, rest, storage, 1)
        B = _solver(nx, ny, faces, rest, storage, 0)
        A.step(17)
        for n in (14, 2, 1):
            B.step(n)
        torch.cuda.synchronize()
        assert torch.equal(A.planes(), B.planes()), (nx, ny, B.run_plan(14)[0])


@pytest.mark.parametrize("nx,ny,faces,rest,storage,kernels", [
    (200000, 2, True, True, "f32", {"step"}),    # tiles: 2.9 times the time of single steps
    (100000, 3, True, True, "f32", {"step"}),    # 2.1
    (20000, 2, False, True, "f32", {"strip"}),   # tiles of 32 x 32: 1.7
    (50000, 2, True, False, "f64", {"strip"}),   # tiles of 64 x 24: 1.4
    (20000, 4, True, False, "f64", {"tile"})])
def test_short_grids_avoid_empty_tiles(nx, ny, faces, rest, storage, kernels):
    plan = _solver(nx, ny, faces, rest, storage, 0).run_plan(48)
    assert {l["kernel"] for l in plan} == kernels
    if kernels == {"tile"}:
        assert max(l["rows"] for l in plan) == 16
