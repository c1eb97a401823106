"""Workgroups of the persistent fused mode: one per compute unit for a small batch, whose
passes a larger grid only closes later; a grid asked for is kept; results do not depend on it."""
import pytest

from gpu_helpers import W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,fuse", [("f64", 8), ("f64", 4), ("f32", 8), ("f32", 7)])
def test_grid_of_a_small_batch(storage, fuse):
    import torch

    from paper_1401_0427_amd.lbm import Batch

    cases = [W.radial_dam_break_2d(n) for n in (40, 64, 130)]
    insts = [dict(dim=2, nx=c.nx, ny=c.ny, lam=c.lam, s=c.s, g=c.g, bc=c.bc, h0=c.h0, qx0=c.qx0, qy0=c.qy0)
             for c in cases]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    runs = []
    for grid, expect in ((0, cus), (cus // 4, cus // 4), (2 * cus, None)):
        B = Batch(insts, storage=storage, mode=4, fuse_steps=fuse, grid=grid)
        assert B.info()[1] == expect or (expect is None and cus <= B.info()[1] <= 2 * cus)
        B.run(19)
        runs.append(B.moments())
    for a, b in zip(runs[0], runs[1]):
        assert torch.equal(a, b)
    for a, b in zip(runs[0], runs[2]):
        assert torch.equal(a, b)
