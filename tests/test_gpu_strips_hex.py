"""The strip kernel of general hexahedra (op_hexs.hip) where its layout can go wrong:
grids at the edges of its bands (3 node rows), blocks (62 columns of the bands laid end
to end) and planes, on meshes with every interior node moved, and the reach of a
non-finite value.  Same bounds as test_gpu_apply.py: FP64 1e-13 of the largest entry,
FP32 64 eps (|A| |x|)_i."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import print_case, to_dev
from test_gpu_apply import jittered_coords

pytestmark = pytest.mark.gpu

EPS32 = np.finfo(np.float32).eps

# cells: the smallest; one band of node rows and one more or less; 62 columns with the
# two past the mesh and one more or less; several bands ending on a block
SIZES = [(1, 1, 1), (2, 1, 3), (5, 2, 2), (5, 3, 1), (4, 5, 2), (60, 3, 2), (61, 2, 1), (59, 5, 2), (29, 8, 1), (14, 17, 9)]


def _scenario(n):
    s = synth.aquifer_hex(ncells=n, n_steps=1)
    s.coords = jittered_coords(s, 0.12, seed=5)
    return s


@pytest.mark.parametrize("n", SIZES, ids=["%dx%dx%d" % n for n in SIZES])
def test_strip_edges(hts, n):
    import torch
    scn = _scenario(n)
    om = oracle.Mesh.of(scn)
    rng = np.random.default_rng(7)
    X, Y, Z = om.coords()
    P = 1e5 + scn.rho_w * scn.g * (scn.extent[2] - Z) - 20.0 * X + 5.0 * rng.standard_normal(om.nnode)
    x = rng.standard_normal(om.nnode)
    m = hts.from_scenario(scn, initial=False)
    m.set_state(0, P, scn.t0)
    rg = scn.rho_w * scn.g
    phi32 = ((P - P[0]) + rg * (Z - Z[0])).astype(np.float32)      # the FP32 operator's pressure
    for field in (0, 1):
        mask, _ = oracle.dirichlet(scn, om, field, scn.t0 + scn.dt)
        for prec in (0, 1):
            print_case("strip hex", n, "field", field, "prec", prec)
            A = oracle.operator(scn, field, P=P if prec == 0 else phi32.astype(np.float64) - rg * (Z - Z[0]) + P[0])
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
    """A NaN or infinity reaches the 27 nodes around it and no other (free rows), or
    its own row alone (a constrained one)."""
    import torch
    n = (61, 9, 5)
    scn = _scenario(n)
    m = hts.from_scenario(scn, initial=True)
    om = oracle.Mesh.of(scn)
    mask = oracle.dirichlet(scn, om, field, scn.t0 + scn.dt)[0].reshape(n[2] + 1, n[1] + 1, n[0] + 1)
    NX, NY, NZ = (v + 1 for v in n)
    for (i, j, k), bad in (((30, 6, 2), np.nan), ((60, 7, 3), np.inf), ((1, 1, 1), np.nan), ((61, 8, 2), np.nan),
                           ((0, 7, 2), np.inf)):
        print_case("non-finite hex", field, prec, (i, j, k), bad)
        x = np.random.default_rng(3).standard_normal((NZ, NY, NX))
        x[k, j, i] = bad
        xd = to_dev(x.reshape(-1), "float64" if prec == 0 else "float32")
        yd = torch.zeros_like(xd)
        m.apply_operator(field, prec, scn.dt, xd, yd)
        off = ~np.isfinite(yd.cpu().numpy().reshape(NZ, NY, NX))
        want = np.zeros_like(off)
        if not mask[k, j, i]:
            want[max(k - 1, 0):k + 2, max(j - 1, 0):j + 2, max(i - 1, 0):i + 2] = True
            want &= ~mask
        want[k, j, i] = True
        assert np.array_equal(off, want)
