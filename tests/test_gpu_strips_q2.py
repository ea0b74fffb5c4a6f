"""The Q2 strip kernel (op_q2s.hip) where its layout can go wrong: grids at the
edges of its bands (3 cell rows for the FP64 heat operator, 7 for the others),
blocks (62 columns of the bands laid end to end) and planes, injection lines that
share a cell column, and the reach of a non-finite value.  Same bounds as
test_gpu_apply.py: FP64 1e-13 of the largest entry, FP32 64 eps (|A| |x|)_i."""
import copy

import numpy as np
import pytest

import oracle
import synth
from gpu_util import print_case, to_dev
from test_gpu_strips import _scenario

pytestmark = pytest.mark.gpu

EPS32 = np.finfo(np.float32).eps

# cells: the smallest; one band of either height and a row more or less; 62 columns
# with the two past the mesh and one more or less; several bands ending on a block
SIZES = [(1, 1, 1), (2, 1, 3), (5, 2, 1), (5, 3, 2), (5, 4, 2), (4, 6, 1), (4, 7, 2), (4, 8, 1), (60, 3, 1), (61, 2, 1),
         (59, 4, 2), (29, 8, 1), (9, 15, 9)]


@pytest.mark.parametrize("graded", [False, True])
@pytest.mark.parametrize("n", SIZES, ids=["%dx%dx%d" % n for n in SIZES])
def test_strip_edges(hts, n, graded):
    import torch
    scn = _scenario(n, graded)
    scn.degree = 2
    om = oracle.Mesh.of(scn)
    rng = np.random.default_rng(7)
    X, Y, Z = om.coords()
    P = 1e5 + scn.rho_w * scn.g * (scn.extent[2] - Z) - 20.0 * X + 5.0 * rng.standard_normal(om.nnode)
    x = rng.standard_normal(om.nnode)
    m = hts.from_scenario(scn, initial=False)
    m.set_state(0, P, scn.t0)
    zk = Z if graded else (np.arange(om.nnode) // (om.dims[0] * om.dims[1])) * (scn.extent[2] / (2 * n[2]))
    rg = scn.rho_w * scn.g
    # the heat operator's reference without its hydrostatic part, P + rho_w g z against
    # no gravity: with it the assembled velocity alone is off by up to 2.3e-13 of the
    # largest entry here (1 m cells under 100 m of water)
    still = copy.deepcopy(scn)
    still.g = 0.0
    PL = np.longdouble(P)
    phi64 = np.asarray((PL - PL[0]) + np.longdouble(rg) * (np.longdouble(Z) - Z[0]), dtype=np.float64)
    phi32 = ((P - P[0]) + rg * zk).astype(np.float32)      # the FP32 operator's pressure
    for field in (0, 1):
        mask, _ = oracle.dirichlet(scn, om, field, scn.t0 + scn.dt)
        for prec in (0, 1):
            print_case("strip q2", n, "graded", graded, "field", field, "prec", prec)
            A = oracle.operator(still if field else scn, field, P=phi64 if prec == 0 else phi32.astype(np.float64))
            ref = oracle.reduced_apply(A, mask, x)
            xd = to_dev(x, "float64" if prec == 0 else "float32")
            yd = torch.zeros_like(xd)
            m.apply_operator(field, prec, scn.dt, xd, yd)
            err = np.abs(yd.double().cpu().numpy() - ref)
            if prec == 0:
                assert err.max() <= 1e-13 * np.abs(ref).max()
            else:
                bound = 64 * EPS32 * (abs(A.tocsr()) @ np.where(mask, 0.0, np.abs(x)))
                assert np.all(err <= np.where(mask, EPS32 * np.abs(x), bound) + 1e-30)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("field", [0, 1])
def test_non_finite_values_stay_local(hts, field, prec):
    """A NaN or infinity reaches the nodes of the cells around it and no other
    (free columns), or its own row alone (a constrained column)."""
    import torch
    n = (31, 9, 3)
    scn = synth.config2(ncells=n, n_steps=1)
    scn.degree = 2
    m = hts.from_scenario(scn, initial=True)
    NX, NY, NZ = (2 * v + 1 for v in n)

    def around(i):
        return slice(i - 2 + i % 2, i + 3 - i % 2)

    for (i, j, k), bad in (((30, 6, 3), np.nan), ((60, 7, 2), np.inf), ((3, 14, 4), np.nan), ((62, 8, 3), np.nan),
                           ((0, 7, 3), np.inf), ((31, 13, 3), np.inf)):
        print_case("non-finite q2", field, prec, (i, j, k), bad)
        x = np.random.default_rng(3).standard_normal((NZ, NY, NX))
        x[k, j, i] = bad
        xd = to_dev(x.reshape(-1), "float64" if prec == 0 else "float32")
        yd = torch.zeros_like(xd)
        m.apply_operator(field, prec, scn.dt, xd, yd)
        off = ~np.isfinite(yd.cpu().numpy().reshape(NZ, NY, NX))
        want = np.zeros_like(off)
        if i in (0, NX - 1):          # on a Dirichlet face of either field
            want[k, j, i] = True
        else:
            want[around(k), around(j), around(i)] = True
            face = np.zeros_like(off)
            face[:, :, [0, -1]] = face[:, [0, -1], :] = True
            if field == 1:
                face[[0, -1]] = True
            want &= ~face
        assert np.array_equal(off, want)
