"""Sums of many partial values: the same bits on every call, near the exact sum;
with faces the partial sums of an adjoint step are one per 256 nodes of a row."""
import math

import pytest

from gpu_helpers import gpu_solver, smooth_random_2d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 4096, 4097, 65537, 262144, 1000003])
def test_sum(n):
    import torch

    S = gpu_solver(smooth_random_2d(20, 20))
    g = torch.Generator().manual_seed(n)
    v = torch.randn(n, generator=g, dtype=torch.float64)
    d = v.cuda()
    first = S.sum(d)
    # pairwise-like order: at most n / 65536 + 18 roundings on any value's way
    assert abs(first - math.fsum(v.tolist())) <= (n / 65536 + 18) * 2.0 ** -53 * float(v.abs().sum())
    S.step(2)
    assert all(S.sum(d) == first for _ in range(4))
    assert S.sum(d[:1]) == float(v[0])


@pytest.mark.parametrize("bc", [("inflow", "neumann", "wall", "inflow"), ("periodic", "periodic", "wall", "wall")])
def test_partials_of_grids_with_faces(bc):
    case = smooth_random_2d(300, 70, bc=bc, inflow={f: (1.1, 0.1, 0.0) for f in range(4) if bc[f] == "inflow"})
    S = gpu_solver(case)
    assert S.adjoint_partials().numel() == 2 * 70
    assert gpu_solver(smooth_random_2d(300, 70)).adjoint_partials().numel() == 75 * 70
