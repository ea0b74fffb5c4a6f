"""Rounding error of operator applies, as a relative 2-norm against extended precision.

A rounded operation on values spread evenly over a binade's logarithm errs by 0.425 u of
its result (root mean square of u / m over 1 <= m < 2; u the unit roundoff).  Of a sum of
box cells one entry sees about 16 roundings of its own size: 3 sums into the modes of the
cell, about 6 in the factor of a mode (cell size, coefficient, their products), its product,
6 sums back into the node.  They are independent, so the bound is 0.425 sqrt(16) u = 1.7 u."""
import numpy as np
import pytest

import synth
from gpu_util import print_case, to_dev

pytestmark = pytest.mark.gpu

LD = np.longdouble
DT, B, MU = 86400.0, 1.0e5, 1.0e-3


def _sum_cells(n, cell):
    """y = sum over the cells: cell(j) gives the 8 corner values (z, y, x) of all cells."""
    y = np.zeros([v + 1 for v in reversed(n)], LD)
    for a in range(8):
        i, j, k = a & 1, a >> 1 & 1, a >> 2
        y[k:k + n[2], j:j + n[1], i:i + n[0]] += cell(a)
    return y


def _corners(u, n):
    return [u[(a >> 2):(a >> 2) + n[2], (a >> 1 & 1):(a >> 1 & 1) + n[1], (a & 1):(a & 1) + n[0]] for a in range(8)]


def _pressure_box(n, edges, k, x):
    """(M + dt B K_k) x of the trilinear cells in extended precision."""
    h = [np.diff(e.astype(LD)) for e in edges]
    hz, hy, hx = np.meshgrid(h[2], h[1], h[0], indexing="ij")
    M, K = np.array([[2, 1], [1, 2]], LD) / 6, np.array([[1, -1], [-1, 1]], LD)
    U, s = _corners(x.reshape([v + 1 for v in reversed(n)]).astype(LD), n), LD(DT) * LD(B) * k.reshape(hx.shape).astype(LD)

    def cell(a):
        out = 0
        for b in range(8):
            m = [M[a >> d & 1, b >> d & 1] for d in range(3)]
            q = [K[a >> d & 1, b >> d & 1] for d in range(3)]
            out = out + U[b] * (m[0] * m[1] * m[2] * (hx * hy * hz) + s * (
                q[0] * m[1] * m[2] * (hy * hz / hx) + m[0] * q[1] * m[2] * (hx * hz / hy) + m[0] * m[1] * q[2] * (hx * hy / hz)))
        return out

    return _sum_cells(n, cell).reshape(-1)


def _edges(length, n, swing):
    s = np.arange(n + 1) / n
    e = length * (s + swing * np.sin(2 * np.pi * s) / (2 * np.pi))
    e[0], e[-1] = 0.0, length
    return e


@pytest.mark.parametrize("graded", [False, True])
@pytest.mark.parametrize("n", [(16, 16, 16), (41, 27, 19)], ids=["16", "41x27x19"])
def test_q1_pressure(hts, n, graded):
    import torch
    ext, rng = (1000.0, 1000.0, 200.0), np.random.default_rng(5)
    nc = n[0] * n[1] * n[2]
    perm = 10.0 ** (-11.0 + 0.5 * rng.standard_normal(nc))
    edges = [_edges(ext[d], n[d], (0.5, 0.4, 0.3)[d]) for d in range(3)] if graded else None
    m = hts.Mesh((0.0, 0.0, 0.0), ext, n, 1, edges=edges)
    m.set_materials(perm, np.full(nc, 0.3), np.full(nc, 2.5), np.full(nc, 2e6), 1000.0, MU, 4.18e6, 0.6, 9.81, B)
    at = edges or [np.arange(n[d] + 1).astype(LD) * (LD(ext[d]) / n[d]) for d in range(3)]
    x32 = rng.standard_normal(m.nnode).astype(np.float32)
    ref = _pressure_box(n, [np.asarray(e, LD) for e in at], perm.astype(LD) / LD(MU), x32)
    for prec, dt, u in ((0, "float64", 2.0 ** -53), (1, "float32", 2.0 ** -24)):
        xd = to_dev(x32, dt)
        yd = torch.zeros_like(xd)
        m.apply_operator(0, prec, DT, xd, yd)
        err = float(np.linalg.norm((yd.cpu().numpy().astype(LD) - ref).astype(np.float64)) / np.linalg.norm(ref.astype(np.float64)))
        print_case("rounding", n, "graded", graded, "prec", prec, "error %.3f u" % (err / u))
        assert err <= 1.7 * u


def _pressure_hex(n, xyz, k, x):
    """(M + dt B K_k) x of trilinear hexahedra at the 2 x 2 x 2 Gauss points in extended precision."""
    shape = [v + 1 for v in reversed(n)]
    X = [_corners(xyz[:, d].reshape(shape).astype(LD), n) for d in range(3)]
    U, s = _corners(x.reshape(shape).astype(LD), n), LD(DT) * LD(B) * k.reshape(list(reversed(n))).astype(LD)
    g = [LD(0.5) - 1 / (2 * np.sqrt(LD(3))), LD(0.5) + 1 / (2 * np.sqrt(LD(3)))]
    out = [0] * 8
    for q in range(8):
        p = [g[q >> d & 1] for d in range(3)]
        one = [[1 - p[d], p[d]] for d in range(3)]
        N = [one[0][a & 1] * one[1][a >> 1 & 1] * one[2][a >> 2] for a in range(8)]
        D = [[(one[0][a & 1] if e != 0 else LD(2 * (a & 1) - 1)) * (one[1][a >> 1 & 1] if e != 1 else LD(2 * (a >> 1 & 1) - 1))
              * (one[2][a >> 2] if e != 2 else LD(2 * (a >> 2) - 1)) for a in range(8)] for e in range(3)]
        J = [[sum(D[e][a] * X[d][a] for a in range(8)) for e in range(3)] for d in range(3)]
        cof = lambda i, j: (J[(i + 1) % 3][(j + 1) % 3] * J[(i + 2) % 3][(j + 2) % 3]
                            - J[(i + 1) % 3][(j + 2) % 3] * J[(i + 2) % 3][(j + 1) % 3])
        C = [[cof(i, j) for j in range(3)] for i in range(3)]
        det = sum(J[0][j] * C[0][j] for j in range(3))
        gr = [sum(D[e][a] * U[a] for a in range(8)) for e in range(3)]
        cg = [sum(C[i][j] * gr[j] for j in range(3)) for i in range(3)]
        h = [sum(C[i][j] * cg[i] for i in range(3)) * (s / det) for j in range(3)]
        u = sum(N[a] * U[a] for a in range(8)) * det
        for a in range(8):
            out[a] = out[a] + (N[a] * u + sum(D[e][a] * h[e] for e in range(3))) / 8
    return _sum_cells(n, lambda a: out[a]).reshape(-1)


@pytest.mark.parametrize("n", [(16, 16, 16), (33, 29, 17)], ids=["16", "33x29x17"])
def test_hexahedra_pressure(hts, n):
    """Here what is rounded at a point averages over the eight: in units of 0.425 u squared
    1.4 (cofactors, determinant, flux) and 3.7 (Jacobian) of these, 1 of the coefficient, 3 of
    the sums into the modes, 9 of the sums back, 18 together: 1.82 u, with the last entries of
    the products 1.85 u."""
    import torch
    ext, rng = (500.0, 500.0, 100.0), np.random.default_rng(5)
    nc = n[0] * n[1] * n[2]
    perm = 10.0 ** (-11.0 + 0.5 * rng.standard_normal(nc))
    xyz = synth.terrain_coords((0.0, 0.0, 0.0), ext, n)
    m = hts.Mesh((0.0, 0.0, 0.0), ext, n, 1, coords=xyz)
    m.set_materials(perm, np.full(nc, 0.3), np.full(nc, 2.5), np.full(nc, 2e6), 1000.0, MU, 4.18e6, 0.6, 9.81, B)
    x32 = rng.standard_normal(m.nnode).astype(np.float32)
    ref = _pressure_hex(n, np.asarray(xyz).reshape(-1, 3), perm.astype(LD) / LD(MU), x32)
    for prec, dt, u in ((0, "float64", 2.0 ** -53), (1, "float32", 2.0 ** -24)):
        xd = to_dev(x32, dt)
        yd = torch.zeros_like(xd)
        m.apply_operator(0, prec, DT, xd, yd)
        err = float(np.linalg.norm((yd.cpu().numpy().astype(LD) - ref).astype(np.float64)) / np.linalg.norm(ref.astype(np.float64)))
        print_case("rounding of hexahedra", n, "prec", prec, "error %.3f u" % (err / u))
        assert err <= 1.85 * u
