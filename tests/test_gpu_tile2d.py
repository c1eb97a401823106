"""2D launches of register tiles (k_tile2d), which default plans take on grids too small
for the wave-strip launches: bit for bit equal to single steps, D2Q4 per component and
D2Q5Q4Q4, both storages, every face rule, at the sizes where the tile shapes change."""
import numpy as np
import pytest

from gpu_helpers import smooth_random_2d

pytestmark = pytest.mark.gpu

RATES = [1.7, 1.6, 1.5, 1.4, 1.8, 1.75, 1.3, 1.65, 1.85, 1.2]
FACES = [("periodic",) * 4, ("inflow", "neumann", "wall", "inflow"),
         ("wall", "inflow", "neumann", "wall"), ("neumann", "wall", "inflow", "neumann"),
         ("periodic", "periodic", "wall", "neumann"), ("neumann", "inflow", "periodic", "periodic")]


def _solver(nx, ny, bc, rest, storage, fuse):
    from paper_1401_0427_amd.lbm import Solver

    inflow = {f: (1.1, 0.15 * (1 - 2 * (f % 2)), 0.05) for f in range(4) if bc[f] == "inflow"}
    c = smooth_random_2d(nx, ny, seed=nx + ny, lam=6.0, s=1.7)
    return Solver(2, nx, ny, lam=c.lam, s=c.s, bc=bc, inflow=inflow, h0=c.h0, qx0=c.qx0,
                  qy0=c.qy0, storage=storage, rest=rest, a=0.05 if rest else 0.0,
                  rates=RATES if rest else None, fuse_steps=fuse)


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("rest", [False, True])
@pytest.mark.parametrize("faces", range(len(FACES)))
def test_tile_launches_equal_single_steps(faces, rest, storage):
    """Grids smaller than one tile (2 x 2: the tile wraps a periodic grid several times),
    one node off a tile's output, long and flat ones, and the first and last sizes of
    every shape; runs of whole launches, an uneven split and a single last step."""
    import torch

    for nx, ny in ((2, 2), (3, 5), (16, 7), (70, 71), (71, 71), (148, 148), (149, 149),
                   (2, 4000), (5000, 3), (300, 299), (301, 299), (301, 300), (391, 383), (570, 575), (633, 631), (640, 640),
                   (1300, 700)):
        steps = 37 if nx * ny < 100000 else 21
        A = _solver(nx, ny, FACES[faces], rest, storage, 1)
        B = _solver(nx, ny, FACES[faces], rest, storage, 0)
        A.step(steps)
        for n in (steps - 14, 13, 1):
            B.step(n)
        torch.cuda.synchronize()
        assert torch.equal(A.planes(), B.planes()), (nx, ny)


def test_tile_launches_keep_the_plan_and_the_checks():
    """The reported plan is that of the grid (one step per launch on a small one), and a
    context that checks its state every 5 steps runs in windows of 5 and still finds a
    diverged state."""
    from paper_1401_0427_amd.lbm import LbmError, Solver

    c = smooth_random_2d(100, 60, seed=3)
    S = Solver(2, 100, 60, lam=6.0, s=1.7, h0=c.h0, qx0=c.qx0, qy0=c.qy0, check_every=5)
    assert S.launch_info()["steps_per_launch"] == 1 and S.launch_plan(7) == [1] * 7
    S.step(23)
    assert S.current()[1] == 23
    S.planes()[0, 3, 4] = np.nan
    with pytest.raises(LbmError):
        S.step(7)
