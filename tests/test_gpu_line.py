"""1D launches with the nodes in registers (k_line: tiles of one wavefront, k_line_whole: a
small domain in one workgroup) against single steps: bit for bit, D1Q2 per component and
D1Q3Q2, both storages, every face rule, at the sizes where the shapes change."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FACES = {"neumann": ("neumann", "neumann"), "inflow-wall": ("inflow", "wall"),
         "wall-inflow": ("wall", "inflow"), "periodic": ("periodic", "periodic")}


def _solver(n, faces, rest, storage, fuse):
    from paper_1401_0427_amd.lbm import Solver

    rng = np.random.default_rng(n)
    x = (np.arange(n) + 0.5) / n
    h0 = np.where(x < 0.5, 1.7, 0.8) + 0.01 * rng.random(n)
    q0 = 0.1 * np.sin(2 * np.pi * x)
    inflow = {f: (1.2, 0.2 - 0.4 * f, 0.0) for f in (0, 1) if FACES[faces][f] == "inflow"}
    return Solver(1, n, 1, lam=8.0 if rest else 4.0, s=1.7, bc=FACES[faces] + ("periodic",) * 2,
                  inflow=inflow, h0=h0, qx0=q0, storage=storage, rest=rest, a=0.1 if rest else 0.0,
                  rates=[1.7, 1.3, 1.9] if rest else None, fuse_steps=fuse)


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("rest", [False, True])
@pytest.mark.parametrize("faces", sorted(FACES))
def test_line_launches_equal_single_steps(faces, rest, storage):
    """Sizes around one lane's nodes, a wavefront (64, 128 nodes), a workgroup (256,
    1024), one tile and several, and enough tiles for one, two and more wavefronts per
    SIMD; runs of several launches and a shorter last one; 300 steps in one launch where
    the domain fits a workgroup."""
    import torch

    for n in (2, 3, 63, 64, 65, 127, 128, 129, 256, 257, 1000, 1024, 1025, 2049, 65537, 270001,
              1 << 20):
        steps = 211 if n <= 70000 else 113
        A = _solver(n, faces, rest, storage, 1)
        A.step(steps)
        for fuse in (0, 16) + ((300,) if n <= 1024 else ()):
            B = _solver(n, faces, rest, storage, fuse)
            B.step(steps - 20)
            B.step(20)
            torch.cuda.synchronize()
            assert torch.equal(A.planes(), B.planes()), (n, fuse)
