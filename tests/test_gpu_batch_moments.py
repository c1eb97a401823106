"""Conserved fields of a batch in one launch: bit for bit those of each instance alone."""
import pytest

from gpu_helpers import W, gpu_solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("block", [64, 256, 512])
def test_batch_moments_equal_each_instance(storage, block):
    """Instances of fewer nodes than a workgroup has threads and of ragged sizes, 1D ones
    (whose qy is zero) among 2D ones."""
    import torch

    from paper_1401_0427_amd.lbm import Batch

    cases = [W.dam_break_1d(37), W.radial_dam_break_2d(9), W.dam_break_1d(700),
             W.radial_dam_break_2d(70), W.dam_break_1d(512), W.radial_dam_break_2d(16)]
    insts = [dict(dim=c.dim, nx=c.nx, ny=c.ny, lam=c.lam, s=c.s, g=c.g, bc=c.bc, h0=c.h0,
                  qx0=c.qx0, qy0=c.qy0 if c.dim == 2 else None) for c in cases]
    B = Batch(insts, storage=storage, block=block, mode=2)
    B.run(11)
    at = 0
    fields = B.moments()
    for c in cases:
        S = gpu_solver(c, storage=storage)
        S.step(11)
        n = c.nx * c.ny
        ref = [f.reshape(-1) for f in S.moments()]
        if c.dim == 1:
            ref.append(torch.zeros_like(ref[0]))
        for got, want in zip(fields, ref):
            assert torch.equal(got[at:at + n], want)
        at += n
