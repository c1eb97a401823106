"""The gradient at a caller's initial fields takes any heights, also those no run starts
from: zero, negative, infinite, subnormal."""
import pytest

from gpu_helpers import W, gpu_solver, smooth_random_2d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [1, 2])
def test_gradient_at_any_heights(dim):
    """Against the same operations in the same order in torch: equal, infinities and NaN
    among them (an infinite height has zero velocity, so its momentum gradient is finite)."""
    import torch

    if dim == 1:
        case = W.dam_break_1d(64)
    else:
        case = smooth_random_2d(8, 8, seed=1)
    S = gpu_solver(case)
    n = 64
    g = torch.Generator().manual_seed(5)
    rnd = lambda *s: torch.randn(*s, generator=g, dtype=torch.float64)
    h = rnd(n).abs() + 0.5
    h[:10] = torch.tensor([0.0, -0.0, float("inf"), -float("inf"), -1.5, 2.0 ** -1030, 2.0 ** 1023.5,
                           2.0 ** -1023, 3e-310, 1e300], dtype=torch.float64)
    qx, qy = rnd(n), rnd(n)
    l = rnd(S.nplanes, n)
    lam = S.new_adjoint()
    S.planes(lam).copy_(l if dim == 1 else l.reshape(-1, 8, 8))
    got = S.adjoint_grad_w0(lam, h.cuda(), qx.cuda(), qy.cuda() if dim == 2 else None)
    ih, c, grav = 1.0 / h, 0.5 / case.lam, case.g
    u = qx * ih
    if dim == 1:
        L = l[2] - l[3]
        ref = [0.5 * (l[0] + l[1]) + c * (grav * h - u * u) * L,
               c * (l[0] - l[1]) + 0.5 * (l[2] + l[3]) + 2.0 * u * c * L]
    else:
        v, gh = qy * ih, grav * h
        L0 = [(l[k] + l[k + 2]) + (l[k + 1] + l[k + 3]) for k in (0, 4, 8)]
        Lx = [l[k] - l[k + 2] for k in (0, 4, 8)]
        Ly = [l[k + 1] - l[k + 3] for k in (0, 4, 8)]
        cross = Ly[1] + Lx[2]
        ref = [0.25 * L0[0] + c * (Lx[1] * (gh - u * u) - cross * (u * v) + Ly[2] * (gh - v * v)),
               c * Lx[0] + 0.25 * L0[1] + c * (2.0 * u * Lx[1] + v * cross),
               c * Ly[0] + 0.25 * L0[2] + c * (2.0 * v * Ly[2] + u * cross)]
    assert torch.isfinite(ref[1][2]) and not torch.isfinite(ref[0][0])
    for a, b in zip(got, ref):
        assert torch.equal(torch.nan_to_num(a.cpu().reshape(-1), nan=12345.0), torch.nan_to_num(b, nan=12345.0))
