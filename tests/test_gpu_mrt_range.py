"""Rest-population runs at heights, and with a g, far outside the usual: bit for bit the
same operations with IEEE divisions, in numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

R1 = [1.7, 1.3, 1.9]
R2 = [1.7, 1.6, 1.5, 1.4, 1.8, 1.75, 1.3, 1.65, 1.85, 1.2]


def _consts(lam, g, a):
    return dict(lam=lam, il=1.0 / lam, a=a, aK=a * (0.5 / g), g=g, hg=0.5 * g, c=0.5 / lam)


def _collide1(f, M, r):
    lam, il = M["lam"], M["il"]
    sp = f[1] + f[2]
    rho = f[0] + sp
    J, eps = lam * (f[1] - f[2]), (lam * lam) * (sp - 2.0 * f[0])
    q, Jq = f[3] + f[4], lam * (f[3] - f[4])
    u, p = q / rho, M["hg"] * (rho * rho)
    theta = M["g"] * rho - 0.5 * (u * u)
    J = J + r[0] * (q - J)
    eps = eps + r[1] * ((lam * lam) * (rho - 3.0 * (M["aK"] * theta)) - eps)
    Jq = Jq + r[2] * ((q * u + p) - Jq)
    f0 = (rho - eps * (il * il)) / 3.0
    S = rho - f0
    return [f0, 0.5 * (S + J * il), 0.5 * (S - J * il), 0.5 * (q + Jq * il), 0.5 * (q - Jq * il)]


def _init1(h, q, M):
    ih = 1.0 / h
    u = q * ih
    f0 = M["aK"] * (M["g"] * h - 0.5 * (u * u))
    hr, F = h - f0, (q * q) * ih + M["hg"] * (h * h)
    return [f0, 0.5 * hr + q * M["c"], 0.5 * hr - q * M["c"], 0.5 * q + F * M["c"], 0.5 * q - F * M["c"]]


def _collide2(f, M, r):
    lam, il = M["lam"], M["il"]

    def moments(g):
        a, b = g[0] + g[2], g[1] + g[3]
        return a + b, lam * (g[0] - g[2]), lam * (g[1] - g[3]), a - b

    def invert(q, mx, my, xx):
        a, b = 0.5 * (q + xx), 0.5 * (q - xx)
        return [0.5 * (a + mx * il), 0.5 * (b + my * il), 0.5 * (a - mx * il), 0.5 * (b - my * il)]

    s13, s24 = f[1] + f[3], f[2] + f[4]
    rho = f[0] + (s13 + s24)
    Jx, Jy = lam * (f[1] - f[3]), lam * (f[2] - f[4])
    eps, XX = (s13 + s24) - 4.0 * f[0], s13 - s24
    qx, fxx, fxy, XXu = moments(f[5:9])
    qy, fyx, fyy, XXv = moments(f[9:13])
    ir = 1.0 / rho
    u, v, p = qx * ir, qy * ir, M["hg"] * (rho * rho)
    Jx, Jy = Jx + r[0] * (qx - Jx), Jy + r[1] * (qy - Jy)
    eps = eps + r[2] * (((1.0 - 2.5 * M["a"]) * rho + (1.25 * M["a"]) * (u * u + v * v) / M["g"]) - eps)
    XX = XX + r[3] * (0.0 - XX)
    fxx, fxy, XXu = fxx + r[4] * ((qx * u + p) - fxx), fxy + r[5] * (qx * v - fxy), XXu + r[6] * (0.0 - XXu)
    fyx, fyy, XXv = fyx + r[7] * (qy * u - fyx), fyy + r[8] * ((qy * v + p) - fyy), XXv + r[9] * (0.0 - XXv)
    f0 = 0.2 * (rho - eps)
    S = rho - f0
    a, b = 0.5 * (S + XX), 0.5 * (S - XX)
    h4 = [0.5 * (a + Jx * il), 0.5 * (b + Jy * il), 0.5 * (a - Jx * il), 0.5 * (b - Jy * il)]
    return [f0] + h4 + invert(qx, fxx, fxy, XXu) + invert(qy, fyx, fyy, XXv)


def _init2(h, qx, qy, M):
    ih = 1.0 / h
    u, v = qx * ih, qy * ih
    f0 = M["aK"] * (M["g"] * h - 0.5 * (u * u + v * v))
    hr, p = h - f0, M["hg"] * (h * h)
    Fxx, Fxy, Fyy = (qx * qx) * ih + p, (qx * qy) * ih, (qy * qy) * ih + p

    def four(z, x, y):
        z, x, y = 0.25 * z, x * M["c"], y * M["c"]
        return [z + x, z + y, z - x, z - y]

    return [f0] + four(hr, qx, qy) + four(qx, Fxx, Fxy) + four(qy, Fxy, Fyy)


@pytest.mark.parametrize("fuse", [0, 16])
@pytest.mark.parametrize("scale", [-1019, -1014, -505])
def test_1d_heights_of_any_size(scale, fuse):
    """Units in which g h is of order one, so the run is an ordinary one."""
    from paper_1401_0427_amd.lbm import Solver

    rng = np.random.default_rng(3)
    n, steps = 300, 40
    h = np.ldexp(1.0 + rng.random(n), scale)
    q = h * (0.3 + 0.2 * rng.random(n))
    S = Solver(1, n, 1, lam=8.0, s=1.7, g=2.0 ** -scale, h0=h, qx0=q, storage="f64", rest=True, a=0.1, rates=R1, fuse_steps=fuse)
    S.step(steps)
    M = _consts(8.0, 2.0 ** -scale, 0.1)
    f = _collide1(_init1(h, q, M), M, R1)
    for _ in range(steps):
        f = _collide1([f[0], np.roll(f[1], 1), np.roll(f[2], -1), np.roll(f[3], 1), np.roll(f[4], -1)], M, R1)
    assert np.all(np.isfinite(f)) and np.array_equal(S.planes().cpu().numpy(), np.stack(f))


@pytest.mark.parametrize("fuse", [0, 5])
@pytest.mark.parametrize("log_g,log_q", [(-1014, -508), (-1018, -511), (0, 0)])
def test_2d_any_g(log_g, log_q, fuse):
    """(0, 0): the usual range, the numpy side checked against the fast launches."""
    from paper_1401_0427_amd.lbm import Solver

    rng = np.random.default_rng(4)
    n, m, steps = 40, 23, 12
    h = 1.0 + 0.2 * rng.random((m, n))
    qx, qy = (np.ldexp(0.1 * (1.0 + rng.random((m, n))), log_q) for _ in range(2))
    g = 2.0 ** log_g * 1.1
    S = Solver(2, n, m, lam=6.0, s=1.7, g=g, h0=h, qx0=qx, qy0=qy, storage="f64", rest=True, a=0.05, rates=R2,
               fuse_steps=fuse)
    S.step(steps)
    M = _consts(6.0, g, 0.05)
    f = _collide2(_init2(h, qx, qy, M), M, R2)
    for _ in range(steps):
        v = [f[0]]
        for k in (1, 5, 9):
            v += [np.roll(f[k], 1, 1), np.roll(f[k + 1], 1, 0), np.roll(f[k + 2], -1, 1), np.roll(f[k + 3], -1, 0)]
        f = _collide2(v, M, R2)
    assert np.all(np.isfinite(f)) and np.array_equal(S.planes().cpu().numpy(), np.stack(f))
