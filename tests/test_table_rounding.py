"""The 1D tables are rounded once: nodes, weights and the lumped mass of a mesh
against the same rules in extended precision.

A Gauss point of a unit cell is (xi + 1) / 2 with xi correctly rounded: 2^-53 of
it and at most two roundings of the map.  An entry of D is a product of three
weights and det J, summed over up to eight cells: at most 12 roundings of 2^-53.
"""
import numpy as np
import pytest

from paper_2512_08571_amd import fehx

R = np.longdouble
EPS = 2.0 ** -53


def _legendre(n, x):
    p0, p1 = np.ones_like(x), x
    for k in range(2, n + 1):
        p0, p1 = p1, ((2 * k - 1) * x * p1 - (k - 1) * p0) / R(k)
    return p1, n * (x * p1 - p0) / (x * x - 1)


def _gauss(n):
    z = -np.cos(R(np.pi) * (np.arange(n, dtype=R) + R(0.75)) / (R(n) + R(0.5)))
    for _ in range(60):
        P, d = _legendre(n, z)
        z = z - P / d
    return z


def _gll(p):
    g = -np.cos(R(np.pi) * np.arange(1, p, dtype=R) / R(p))
    for _ in range(60):
        P, d = _legendre(p, g)
        g = g - d / ((2 * g * d - p * (p + R(1)) * P) / (1 - g * g))
    P = np.concatenate([[R(1)], _legendre(p, g)[0], [R(1)]])
    return 2 / (p * (p + R(1)) * P * P)


@pytest.mark.parametrize("dq", [0, 2, 3])
@pytest.mark.parametrize("p", range(2, 9))
def test_points_and_lumped_mass(p, dq):
    nq = p + 1 + dq
    m = fehx.Mesh(np.diag([2.0, 2.0, 2.0]), (2, 2, 2), p, nq, (0, 0, 0), device=-1)
    x = m.quad_points().reshape(8, nq, nq, nq, 3)[0, 0, 0, :, 0].astype(R)
    want = (_gauss(nq) + 1) / 2
    assert float(np.abs(x - want).max()) <= 3 * EPS
    w = _gll(p) / 2
    one = np.concatenate([[2 * w[0]], w[1:p]])
    one = np.concatenate([one, one])                      # two cells of a periodic axis
    want = (one[:, None, None] * one[None, :, None] * one[None, None, :]).reshape(-1)
    D = m.lumped_mass().astype(R)
    assert float((np.abs(D - want) / want).max()) <= 12 * EPS
