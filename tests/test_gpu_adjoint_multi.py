"""Adjoint sweeps that run several steps per launch (tiles over stored levels on small
all-periodic grids, two-step strips on larger ones) and the launches that store every
level: bit for bit what one-step launches give, states, adjoints and dL/ds partials."""
import numpy as np
import pytest

from gpu_helpers import gpu_solver, smooth_random_2d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,adj", [("f64", None), ("f32", "f32"), ("f32", "f64")])
@pytest.mark.parametrize("nx,ny", [(2, 2), (3, 7), (57, 16), (109, 110), (110, 110), (223, 224), (250, 251),
                                   (316, 317), (370, 375), (450, 444), (547, 548), (548, 548), (56, 6000),
                                   (6001, 57), (840, 834), (1450, 1400)])
def test_sweeps_equal_single_steps(nx, ny, storage, adj):
    """The first and last sizes of every shape (tiles of 16^2 .. 32^2 nodes, strips of 56
    and 48 columns with a ragged last one and uneven segments), grids smaller than a tile, and
    segment lengths with every remainder."""
    import torch

    case = smooth_random_2d(nx, ny, seed=nx % 7, lam=6.0, s=1.7)
    S = gpu_solver(case, storage=storage, adjoint_storage=adj)
    S.step(3)
    ck = S.current()[0].clone()
    nb = S.nplanes * S.ps
    rng = np.random.default_rng(1)
    lam_T = torch.as_tensor(rng.standard_normal(nb), device="cuda").to(S.adj_dtype)

    def planes(t):
        return t.as_strided((12, ny, nx), (S.ps, nx, 1))

    for n in (2, 5, 8, 11) if nx * ny < 200000 else (6, 9):
        states = [ck]
        for _ in range(n):
            nxt = S.new_state()
            S.step_buffers(states[-1], nxt)
            states.append(nxt)
        a, b, pa = lam_T.clone(), S.new_adjoint(), S.adjoint_partials()
        for t in range(n - 1, -1, -1):
            S.adjoint_step(states[t], a, b, pa)
            a, b = b, a
        la, lb, pb = lam_T.clone(), S.new_adjoint(), S.adjoint_partials()
        out = S.adjoint_segment(ck, n, S.new_state(n - 1), la, lb, pb)
        assert out == n % 2
        assert torch.equal(planes(lb if out else la), planes(a)) and torch.equal(pa, pb), n
        levels = S.new_state(n)
        S.step_levels(ck, n, levels)
        for i in range(n):
            assert torch.equal(planes(levels[i * nb:(i + 1) * nb]), planes(states[i + 1])), (n, i)
        la, lb, pb = lam_T.clone(), S.new_adjoint(), S.adjoint_partials()
        out = S.adjoint_levels(torch.cat(states[:n]), n, la, lb, pb)
        assert out == n % 2
        assert torch.equal(planes(lb if out else la), planes(a)) and torch.equal(pa, pb), n
        # the sum over many groups, in two launches, against a plain one
        got, ref = S.sum(pa), float(pa.sum())
        assert abs(got - ref) <= 1e-13 * float(pa.abs().sum())


@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_levels_with_faces_equal_single_steps(storage):
    """Every level stored on grids with inflow, Neumann and wall faces."""
    import torch

    for nx, ny in ((35, 20), (200, 160), (400, 390), (700, 640)):
        case = smooth_random_2d(nx, ny, seed=2, bc=("inflow", "neumann", "wall", "inflow"),
                                inflow={0: (1.1, 0.15, 0.05), 3: (1.0, 0.1, -0.1)})
        S = gpu_solver(case, storage=storage)
        nb = S.nplanes * S.ps
        prev = S.current()[0].clone()
        levels = S.new_state(11)
        S.step_levels(prev, 11, levels)
        for i in range(11):
            nxt = S.new_state()
            S.step_buffers(prev, nxt)
            assert torch.equal(S.planes(nxt), S.planes(levels[i * nb:(i + 1) * nb])), (nx, i)
            prev = nxt
