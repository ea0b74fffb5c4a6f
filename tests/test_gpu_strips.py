"""The Q1 strip kernel (op_q1s.hip) where its layout can go wrong: grids at the
edges of its bands (7 node rows), blocks (62 node columns of the bands laid end
to end) and planes, injection lines that share a cell column, and the reach of a
non-finite value.  Same bounds as test_gpu_apply.py: FP64 1e-13 of the largest
entry (rounding of a ~200-term sum), FP32 64 eps (|A| |x|)_i."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import print_case, to_dev

pytestmark = pytest.mark.gpu

EPS32 = np.finfo(np.float32).eps

# cells: the smallest; one band and a row more or less; 62 columns with the
# empty one and one more or less; several bands whose columns end on a block
SIZES = [(1, 1, 1), (2, 1, 3), (5, 5, 1), (5, 6, 2), (5, 7, 2), (60, 6, 2), (61, 6, 1), (59, 6, 3), (29, 13, 2),
         (123, 7, 1), (14, 27, 17)]


def _scenario(n, graded):
    s = synth.config2(ncells=n, n_steps=1)
    # a second injection line in the first one's cell column, and one on a
    # node column over part of the height
    s.lines = list(s.lines) + [synth.LineSource(151.0, 251.0, 10.0, 90.0, synth.LINE_WELL, synth.timefn(0.004), 300.0),
                               synth.LineSource(250.0, 250.0, 33.0, 77.0, synth.LINE_WELL, synth.timefn(0.007), 310.0)]
    if graded:
        s.edges = tuple(synth.graded_edges(0.0, s.extent[d], n[d], [(0.3 * s.extent[d], 0.6 * s.extent[d])])
                        for d in range(3))
    return s


@pytest.mark.parametrize("graded", [False, True])
@pytest.mark.parametrize("n", SIZES, ids=["%dx%dx%d" % n for n in SIZES])
def test_strip_edges(hts, n, graded):
    import torch
    scn = _scenario(n, graded)
    om = oracle.Mesh.of(scn)
    rng = np.random.default_rng(7)
    X, Y, Z = om.coords()
    P = 1e5 + scn.rho_w * scn.g * (scn.extent[2] - Z) - 20.0 * X + 5.0 * rng.standard_normal(om.nnode)
    x = rng.standard_normal(om.nnode)
    m = hts.from_scenario(scn, initial=False)
    m.set_state(0, P, scn.t0)
    zk = Z if graded else (np.arange(om.nnode) // (om.dims[0] * om.dims[1])) * (scn.extent[2] / n[2])
    rg = scn.rho_w * scn.g
    phi32 = ((P - P[0]) + rg * zk).astype(np.float32)      # the FP32 operator's pressure
    for field in (0, 1):
        mask, _ = oracle.dirichlet(scn, om, field, scn.t0 + scn.dt)
        for prec in (0, 1):
            print_case("strip", n, "graded", graded, "field", field, "prec", prec)
            A = oracle.operator(scn, field, P=P if prec == 0 else phi32.astype(np.float64) - rg * zk + P[0])
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


@pytest.mark.parametrize("field", [0, 1])
def test_non_finite_values_stay_local(hts, field):
    """A NaN or infinity reaches the 27 nodes around it and no other (free
    columns), or its own row alone (a constrained column)."""
    import torch
    n = (61, 13, 5)
    scn = synth.config2(ncells=n, n_steps=1)
    m = hts.from_scenario(scn, initial=True)
    NX, NY, NZ = (v + 1 for v in n)
    for (i, j, k), bad in (((30, 6, 2), np.nan), ((60, 7, 3), np.inf), ((1, 1, 1), np.nan), ((61, 8, 2), np.nan),
                           ((0, 7, 2), np.inf)):
        print_case("non-finite", field, (i, j, k), bad)
        x = np.random.default_rng(3).standard_normal((NZ, NY, NX))
        x[k, j, i] = bad
        xd = to_dev(x.reshape(-1))
        yd = torch.zeros_like(xd)
        m.apply_operator(field, 0, scn.dt, xd, yd)
        off = ~np.isfinite(yd.cpu().numpy().reshape(NZ, NY, NX))
        want = np.zeros_like(off)
        if i in (0, NX - 1):          # on a Dirichlet face of either field
            want[k, j, i] = True
        else:
            want[k - 1:k + 2, j - 1:j + 2, i - 1:i + 2] = True
            face = np.zeros_like(off)
            face[:, :, [0, -1]] = face[:, [0, -1], :] = True
            if field == 1:
                face[[0, -1]] = True
            want &= ~face
        assert np.array_equal(off, want)
